// a1: cell binning, stable sort of the cell keys, cell ranges, the
// list of occupied bricks and the gather of granule arrays into sorted order
// (gfx950).
//
// The contact test of Sec. 3.1 only pairs granules closer than r_i + r_j;
// binning granules into cells of edge >= 2 r_max and sorting them by cell
// makes each granule's candidates the occupants of at most 27 cells, stored
// contiguously so that later stages read them coalesced.
//
// The keys are cells, so most sorts count: every granule takes a place in its
// cell with an atomic on the cell's counter, a scan of the counters gives the
// cell ranges (needed in any case), and the granules of each cell are then
// put in input order, which makes the sort stable whatever order the atomics
// ran in.  Six launches for any number of cells (keys, counts, two scan
// passes, places, order; one scan pass fewer for small tables).  Cells of many
// granules and large shuffled inputs are sorted by passes over 8-bit digits, three
// launches each, whose cost does not depend on the input (see sort_limit).
#include "gic_launch.hpp"

namespace gic {

namespace {

// Key of every granule; flags non-finite and out-of-box positions.  With
// the previous sorted keys pk (same n), granules whose key differs from
// pk at their position are appended to chg (up to kChgCap; ctl[0] counts
// them all).  With xref (the positions of the neighbour list's build, same
// order), each workgroup writes the largest squared displacement of its
// granules since the build to dpart[block] (no atomics: one address hit by
// every wave would serialise them).  With pk the order and the sorted keys of
// an unchanged state (the identity and the keys themselves) are written here,
// so that a sort that finds no changed key has nothing left to write.
__global__ void __launch_bounds__(256) k_cell_keys(DevParams P, int64_t n, const double *__restrict__ x,
                                                   uint32_t *__restrict__ key, int64_t *err,
                                                   const uint32_t *__restrict__ pk, uint64_t *__restrict__ chg,
                                                   int32_t *__restrict__ ctl, const float *__restrict__ xref,
                                                   float *__restrict__ dpart, int32_t *__restrict__ order,
                                                   uint32_t *__restrict__ skeys)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (xref) {
        float d2 = 0.0f;
        if (i < n) {
            double s2 = 0.0;
            for (int a = 0; a < 3; ++a) {
                const double d = x[a * n + i] - (double)xref[a * n + i];
                s2 += d * d;
            }
            d2 = (float)s2;
            if (!(d2 >= 0.0f)) d2 = __builtin_huge_valf();  // NaN: rebuild (the position is flagged below)
        }
        __shared__ float s_d2[4];
        for (int off = 32; off > 0; off >>= 1) d2 = fmaxf(d2, __shfl_xor(d2, off));
        if ((threadIdx.x & 63) == 0) s_d2[threadIdx.x >> 6] = d2;
        __syncthreads();
        if (threadIdx.x == 0) dpart[blockIdx.x] = fmaxf(fmaxf(s_d2[0], s_d2[1]), fmaxf(s_d2[2], s_d2[3]));
    }
    bool changed = false;
    uint32_t k = 0;
    if (i < n) {
        double xa[3] = {x[i], x[n + i], x[2 * n + i]};
        int32_t c[3];
        bool bad = false, out = false;
        for (int a = 0; a < 3; ++a) {
            bad |= !isfinite(xa[a]);
            out |= !(xa[a] >= 0.0 && xa[a] < P.L[a]);
            c[a] = cell_coord(xa[a], P.inv_cell, P.nc[a]);
        }
        if (bad) raise_error(err, kErrNonFinite, i);
        else if (out) raise_error(err, kErrDomain, i);
        k = key_of_cell(P, c[0], c[1], c[2]);
        key[i] = k;
        if (pk) {
            changed = pk[i] != k;
            order[i] = (int32_t)i;
            skeys[i] = k;
        }
    }
    if (!pk) return;
    // changed keys appended with one counter atomic per workgroup that has
    // any (a moving bed changes many keys, and atomics on one address
    // serialise: one per wave cost 11 us on 65,536 granules)
    __shared__ int32_t s_cnt[4];
    __shared__ int32_t s_base;
    const uint64_t mask = __ballot(changed);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) s_cnt[wave] = (int32_t)__popcll(mask);
    __syncthreads();
    const int32_t tot = s_cnt[0] + s_cnt[1] + s_cnt[2] + s_cnt[3];
    if (tot == 0) return;
    if (threadIdx.x == 0) s_base = atomicAdd(&ctl[0], tot);
    __syncthreads();
    if (changed) {
        int32_t slot = s_base + (int32_t)__popcll(mask & ((1ull << lane) - 1ull));
        for (int w = 0; w < wave; ++w) slot += s_cnt[w];
        if (chg && slot < kChgCap) chg[slot] = ((uint64_t)k << 32) | (uint64_t)i;
    }
}

// Exclusive prefix sum in place, in three coalesced phases: each workgroup
// reduces one contiguous chunk, one workgroup scans the chunk totals, then
// each workgroup rescans its chunk 1024 entries at a time from its offset.
constexpr int kScanThreads = 1024;

__device__ inline uint32_t block_reduce_sum(uint32_t v, uint32_t *lds)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) lds[wave] = v;
    __syncthreads();
    uint32_t t = 0;
    if (threadIdx.x < 64) {
        t = threadIdx.x < (blockDim.x >> 6) ? lds[threadIdx.x] : 0u;
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off);
    }
    __syncthreads();
    return t;  // valid in wave 0
}

// Inclusive scan over the workgroup (thread order); *total = sum of all.
__device__ inline uint32_t block_scan_inclusive(uint32_t v, uint32_t *lds, uint32_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int off = 1; off < 64; off <<= 1) {
        uint32_t t = __shfl_up(v, off);
        if (lane >= off) v += t;
    }
    if (lane == 63) lds[wave] = v;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int nw = blockDim.x >> 6;
        uint32_t w = threadIdx.x < nw ? lds[threadIdx.x] : 0u;
        for (int off = 1; off < 64; off <<= 1) {
            uint32_t t = __shfl_up(w, off);
            if (lane >= off) w += t;
        }
        if (threadIdx.x < nw) lds[threadIdx.x] = w;  // inclusive prefix of wave totals
    }
    __syncthreads();
    const uint32_t before = wave > 0 ? lds[wave - 1] : 0u;
    *total = lds[(blockDim.x >> 6) - 1];
    __syncthreads();
    return v + before;
}

// The sum over t < m of a[t] (m <= kScanThreads), in every thread.
__device__ inline uint32_t prefix_before(const uint32_t *__restrict__ a, int m, uint32_t *lds)
{
    __shared__ uint32_t s_sum;
    const uint32_t v = block_reduce_sum((int)threadIdx.x < m ? a[threadIdx.x] : 0u, lds);
    if (threadIdx.x == 0) s_sum = v;
    __syncthreads();
    const uint32_t r = s_sum;
    __syncthreads();
    return r;
}

// First scan pass over the cell counts: each chunk's granules (sums) and
// occupied bricks (bsums).  A brick is 64 consecutive keys, four per lane of
// sixteen lanes.  skip (optional): the sort's control words; skip[2] set means the cell
// ranges and bricks of the last sort still hold (no key changed).
__global__ void __launch_bounds__(kScanThreads) k_scan_reduce(const uint32_t *__restrict__ a, int64_t len,
                                                              int64_t chunk, uint32_t *__restrict__ sums,
                                                              uint32_t *__restrict__ bsums,
                                                              const int32_t *__restrict__ skip)
{
    if (skip && skip[2]) return;
    __shared__ uint32_t lds[kScanThreads / 64];
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < len ? lo + chunk : len;
    uint32_t s = 0, nb = 0;
    const int lane = threadIdx.x & 63;
    for (int64_t k = lo + 4 * (int64_t)threadIdx.x; k < hi; k += 4 * kScanThreads) {  // len: a multiple of 64
        const uint4 v = *reinterpret_cast<const uint4 *>(a + k);
        const uint32_t t = ((v.x + v.y) + v.z) + v.w;
        s += t;
        const uint64_t m = __ballot(t != 0u);
        if ((lane & 15) == 0) nb += (m >> lane) & 0xFFFFull ? 1u : 0u;
    }
    s = block_reduce_sum(s, lds);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
    nb = block_reduce_sum(nb, lds);
    if (threadIdx.x == 0) bsums[blockIdx.x] = nb;
}

// Lanes of a wave from this one up to the next lane of `starts` (a run).
__device__ inline int run_length(uint64_t starts)
{
    const int lane = threadIdx.x & 63;
    const uint64_t above = lane == 63 ? 0ull : (starts >> (lane + 1)) << (lane + 1);
    return (above ? __ffsll((unsigned long long)above) - 1 : 64) - lane;
}

__device__ inline int lower_bound_u64(const uint64_t *a, int m, uint64_t v)
{
    int lo = 0, hi = m;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ inline int lower_bound_u32(const uint32_t *a, int m, uint32_t v)
{
    int lo = 0, hi = m;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (a[mid] < v) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Counts of the cells, and each granule's place in its cell in order of
// arrival (slot): one atomic per run of equal keys inside a wave.  After an
// incremental sort (ctl[1]) no places are needed: the granules that kept
// their key (U, see k_chg_sort) and are displaced by those that did not are
// written to order and skeys instead.  Small sorts (one launch fewer: chg not
// collected) decide here (decide 1): the first workgroup writes ctl[2] (no key
// changed) and, with nl, whether the neighbour list must be rebuilt.  Sorts by
// digits (decide 2) count here after the incremental path only.
__global__ void __launch_bounds__(256) k_cell_count(const uint32_t *__restrict__ key, int64_t n,
                                                    uint32_t *__restrict__ cnt, uint32_t *__restrict__ slot,
                                                    const uint32_t *__restrict__ pk, const uint64_t *__restrict__ chg_s,
                                                    const uint32_t *__restrict__ chg_p, uint32_t *__restrict__ skeys,
                                                    int32_t *__restrict__ order, int32_t *__restrict__ ctl, int decide,
                                                    int keep, uint32_t *__restrict__ nl, int force, float thr2,
                                                    const float *__restrict__ dpart, int64_t nd)
{
    bool same = false, inc = false;
    const int m = ctl ? ctl[0] : 0;
    if (decide == 1) {
        same = m == 0;
        if (blockIdx.x == 0) {
            __shared__ float s_dm[4];
            float dm = 0.0f;
            if (dpart)
                for (int64_t i = threadIdx.x; i < nd; i += 256) dm = fmaxf(dm, dpart[i]);
            for (int off = 32; off > 0; off >>= 1) dm = fmaxf(dm, __shfl_xor(dm, off));
            if ((threadIdx.x & 63) == 0) s_dm[threadIdx.x >> 6] = dm;
            __syncthreads();
            if (threadIdx.x == 0) {
                const float d2 = fmaxf(fmaxf(s_dm[0], s_dm[1]), fmaxf(s_dm[2], s_dm[3]));
                ctl[1] = 0;
                ctl[2] = same ? 1 : 0;
                if (nl) nl[0] = (force || m != 0 || !(d2 < thr2)) ? 1u : 0u;
            }
        }
    } else if (ctl) {
        inc = ctl[1] != 0;
        same = ctl[2] != 0;
    }
    if ((same && keep) || (decide == 2 && !inc)) return;
    const int lane = threadIdx.x & 63;
    for (int64_t q0 = (int64_t)blockIdx.x * 256; q0 < n; q0 += (int64_t)gridDim.x * 256) {
        const int64_t q = q0 + threadIdx.x;
        const bool valid = q < n;
        const uint32_t k = valid ? key[q] : 0u;
        const uint32_t before = __shfl_up(k, 1);
        // run heads; invalid lanes end the last run
        const uint64_t starts = __ballot(valid && (lane == 0 || before != k)) | (~__ballot(valid));
        const bool first = valid && ((starts >> lane) & 1ull);
        uint32_t at = 0;
        if (first) at = atomicAdd(&cnt[k], (uint32_t)run_length(starts));
        if (inc) {
            if (same || !valid || k != pk[q]) continue;  // a changed element: placed by k_chg_sort
            const int64_t place = q - lower_bound_u32(chg_p, m, (uint32_t)q) +
                                  lower_bound_u64(chg_s, m, ((uint64_t)k << 32) | (uint64_t)q);
            if (place == q) continue;  // written by the key kernel
            order[place] = (int32_t)q;
            skeys[place] = k;
            continue;
        }
        const uint64_t upto = starts & (~0ull >> (63 - lane));  // run heads at or below this lane
        const int head = upto ? 63 - __clzll((long long)upto) : 0;
        at = __shfl(at, head) + (uint32_t)(lane - head);
        if (valid) slot[q] = at;
    }
}

// Second scan pass: begin = exclusive prefix, end = inclusive prefix of the
// cell counts; the list of occupied bricks in brick order and each brick's
// place in it.  A workgroup adds up what lies before its chunk itself: the
// chunk sums of the first pass (at most 1,024 words), or, for tables of at
// most kDirectScan cells, which then have no first pass, the counts (the
// counts are reset to zero for the next sort by k_cell_order).
constexpr int64_t kDirectScan = 32768;

// A list's count and the granules it is of (BrickSeen); of another number than the
// list before, nothing else is known yet (a sort says itself how many keys changed).
// n < 0: a list whose caller does not know, no record.
__device__ inline void put_count(int32_t *count, int32_t nocc, int32_t n, bool sorted)
{
    count[0] = nocc;
    if (n < 0) return;
    if (count[1] != n) {
        count[2] = count[3] = 0;
        if (!sorted) count[4] = n;
        count[5] = -1;
    }
    count[1] = n;
}

__global__ void __launch_bounds__(kScanThreads) k_scan_down_ranges(uint32_t *__restrict__ cnt,
                                                                   uint32_t *__restrict__ begin,
                                                                   uint32_t *__restrict__ end, int64_t len,
                                                                   int64_t chunk, const uint32_t *__restrict__ sums,
                                                                   const uint32_t *__restrict__ bsums,
                                                                   int32_t *__restrict__ ctl, int keep,
                                                                   int32_t *__restrict__ list,
                                                                   int32_t *__restrict__ count,
                                                                   int32_t *__restrict__ slot_of, int32_t n,
                                                                   int compared)
{
    if (keep && ctl[2]) return;  // ranges unchanged (and no changed granule to uncount)
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        count[4] = compared ? ctl[0] : n;
        ctl[0] = 0;  // no changed granules counted for the next sort
    }
    __shared__ uint32_t lds[kScanThreads / 64];
    __shared__ uint32_t s_occ[kScanThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = lo + chunk < len ? lo + chunk : len;
    uint32_t carry, nocc;
    if (sums) {
        carry = prefix_before(sums, (int)blockIdx.x, lds);
        nocc = prefix_before(bsums, (int)blockIdx.x, lds);
    } else {
        // four cells per lane, sixteen lanes per brick, all loads in flight
        constexpr int kBatch = (int)(kDirectScan / (4 * kScanThreads));
        uint32_t a = 0, b = 0;
        const uint4 *c4 = reinterpret_cast<const uint4 *>(cnt);
        const int groups = (int)(lo / (4 * kScanThreads));  // chunks are whole groups
        uint4 v[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            v[u] = u < groups ? c4[(int64_t)u * kScanThreads + threadIdx.x] : uint4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t t = ((v[u].x + v[u].y) + v[u].z) + v[u].w;
            a += t;
            const uint64_t m = __ballot(t != 0u);
            if ((lane & 15) == 0) b += (m >> lane) & 0xFFFFull ? 1u : 0u;
        }
        __shared__ uint32_t s_before[2];
        a = block_reduce_sum(a, lds);
        b = block_reduce_sum(b, lds);
        if (threadIdx.x == 0) {
            s_before[0] = a;
            s_before[1] = b;
        }
        __syncthreads();
        carry = s_before[0];
        nocc = s_before[1];
    }
    // four cells per lane, so sixteen lanes per brick and four bricks per wave
    for (int64_t base = lo; base < hi; base += 4 * kScanThreads) {
        const int64_t k = base + 4 * (int64_t)threadIdx.x;
        uint4 *c4 = reinterpret_cast<uint4 *>(cnt + k);
        const uint4 v = k < hi ? *c4 : uint4{0u, 0u, 0u, 0u};
        const uint32_t t = ((v.x + v.y) + v.z) + v.w;
        const uint64_t m = __ballot(t != 0u);
        const uint32_t occ = ((m & 0xFFFFull) ? 1u : 0u) | ((m & 0xFFFF0000ull) ? 2u : 0u) |
                             ((m & 0xFFFF00000000ull) ? 4u : 0u) | ((m & 0xFFFF000000000000ull) ? 8u : 0u);
        if (lane == 0) s_occ[wave] = __popc(occ);
        uint32_t total;
        const uint32_t before = carry + block_scan_inclusive(t, lds, &total) - t;  // (its barriers also publish s_occ)
        uint32_t place = nocc;
        for (int w = 0; w < kScanThreads / 64; ++w) {
            if (w < wave) place += s_occ[w];
            nocc += s_occ[w];
        }
        if (k < hi) {
            const uint32_t e0 = before + v.x, e1 = e0 + v.y, e2 = e1 + v.z, e3 = e2 + v.w;
            begin[k] = before;
            begin[k + 1] = e0;
            begin[k + 2] = e1;
            begin[k + 3] = e2;
            end[k] = e0;
            end[k + 1] = e1;
            end[k + 2] = e2;
            end[k + 3] = e3;
            if (sums && t != 0u) *c4 = uint4{0u, 0u, 0u, 0u};
            if ((lane & 15) == 0) {
                const int64_t b = k >> 6;
                const int g = lane >> 4;
                const uint32_t at = place + __popc(occ & ((1u << g) - 1u));
                const bool mine = (occ >> g) & 1u;
                if (mine) list[at] = (int32_t)b;
                slot_of[b] = mine ? (int32_t)at : -1;
            }
        }
        carry += total;
        __syncthreads();  // s_occ is rewritten by the next round
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) put_count(count, (int32_t)nocc, n, true);
}

// Granule i to its place in its cell, in order of arrival; the key of the
// place is final.
__global__ void __launch_bounds__(256) k_cell_place(const uint32_t *__restrict__ key, int64_t n,
                                                    const uint32_t *__restrict__ begin,
                                                    const uint32_t *__restrict__ slot, int32_t *__restrict__ tmp,
                                                    uint32_t *__restrict__ skeys, const int32_t *__restrict__ ctl,
                                                    int keep)
{
    if (ctl && (ctl[1] || (keep && ctl[2]))) return;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const uint32_t k = key[i];
        const int64_t p = (int64_t)begin[k] + slot[i];
        if (p >= n) continue;
        tmp[p] = (int32_t)i;
        skeys[p] = k;
    }
}

// Rank of each lane's digit among the lanes of its wave with the same digit
// (8 ballots), and the number of such lanes.
__device__ inline uint64_t digit_mask(uint32_t d, bool valid)
{
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        m &= bit ? bb : ~bb;
    }
    return m;
}

// ---- digit passes (count, scan, scatter) ----------------------------------
//
// Each 8-bit digit pass is three kernels with no waits between workgroups: every
// tile of keys counts its digits (k_digit_count, into tcnt[digit][tile]); one
// workgroup per digit turns its row into the exclusive prefix over the tiles
// and records the row's total (k_digit_scan); every tile then scatters its keys
// stably (k_digit_scatter) from the prefix of its tile plus the keys of all
// smaller digits (a scan of the 256 row totals).  skip (optional): the sort's
// control words; skip[1] set means the incremental path sorted this time.
constexpr int64_t kDigitGrid = 1024;  // workgroups of the tile loops

template <int ITEMS>
__global__ void __launch_bounds__(kSortThreads) k_digit_count(const uint32_t *__restrict__ kin, int64_t n, int pass,
                                                              int64_t tiles, uint32_t *__restrict__ tcnt,
                                                              const int32_t *__restrict__ skip)
{
    if (skip && skip[1]) return;
    __shared__ uint32_t s_cnt[256];
    const int tid = threadIdx.x, lane = tid & 63, shift = 8 * pass;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        s_cnt[tid] = 0;
        __syncthreads();
        const int64_t tile0 = t * (kSortThreads * ITEMS);
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int64_t p = tile0 + (int64_t)it * kSortThreads + tid;
            const bool valid = p < n;
            const uint32_t d = valid ? (kin[p] >> shift) & 255u : 0u;
            const uint64_t m = digit_mask(d, valid);
            if (valid && (m & lt) == 0) atomicAdd(&s_cnt[d], (uint32_t)__popcll(m));
        }
        __syncthreads();
        tcnt[(int64_t)tid * tiles + t] = s_cnt[tid];
        __syncthreads();
    }
}

// Thread i of a row's workgroup takes a contiguous chunk, so the row is read in
// one sweep and scanned once.
__global__ void __launch_bounds__(kSortThreads) k_digit_scan(uint32_t *__restrict__ tcnt, int64_t tiles,
                                                             uint32_t *__restrict__ rowtot,
                                                             const int32_t *__restrict__ skip)
{
    if (skip && skip[1]) return;
    __shared__ uint32_t lds[kSortThreads / 64];
    uint32_t *row = tcnt + (int64_t)blockIdx.x * tiles;
    const int64_t chunk = (tiles + kSortThreads - 1) / kSortThreads;
    const int64_t lo = (int64_t)threadIdx.x * chunk, hi = lo + chunk < tiles ? lo + chunk : tiles;
    uint32_t sum = 0;
    for (int64_t t = lo; t < hi; ++t) sum += row[t];
    uint32_t total;
    uint32_t run = block_scan_inclusive(sum, lds, &total) - sum;
    for (int64_t t = lo; t < hi; ++t) {
        const uint32_t c = row[t];
        row[t] = run;
        run += c;
    }
    if (threadIdx.x == 0) rowtot[blockIdx.x] = total;
}

// Keys and values (vin, or the positions), in rounds of 256 in position order.
template <int ITEMS>
__global__ void __launch_bounds__(kSortThreads) k_digit_scatter(const uint32_t *__restrict__ kin,
                                                                const int32_t *__restrict__ vin,
                                                                uint32_t *__restrict__ kout, int32_t *__restrict__ vout,
                                                                int64_t n, int pass, int64_t tiles,
                                                                const uint32_t *__restrict__ tcnt,
                                                                const uint32_t *__restrict__ rowtot,
                                                                const int32_t *__restrict__ skip)
{
    if (skip && skip[1]) return;
    __shared__ uint32_t s_base[256];  // where this tile's next key of each digit goes
    __shared__ uint32_t wcnt[kSortThreads / 64][256];
    __shared__ uint32_t lds[kSortThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, shift = 8 * pass;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int w = 0; w < kSortThreads / 64; ++w) wcnt[w][tid] = 0;
    const uint32_t g = rowtot[tid];
    uint32_t total;
    const uint32_t dbase = block_scan_inclusive(g, lds, &total) - g;  // keys of all smaller digits
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t tile0 = t * (kSortThreads * ITEMS);
        uint32_t k[ITEMS];
        int32_t val[ITEMS];
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int64_t p = tile0 + (int64_t)it * kSortThreads + tid;
            const bool valid = p < n;
            k[it] = valid ? kin[p] : 0xffffffffu;
            val[it] = valid ? (vin ? vin[p] : (int32_t)p) : 0;
        }
        s_base[tid] = dbase + tcnt[(int64_t)tid * tiles + t];
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITEMS; ++it) {
            const int64_t p = tile0 + (int64_t)it * kSortThreads + tid;
            const bool valid = p < n;
            const uint32_t d = (k[it] >> shift) & 255u;
            const uint64_t m = digit_mask(d, valid);
            const uint32_t rank = (uint32_t)__popcll(m & lt);
            if (valid && rank == 0) wcnt[wave][d] = (uint32_t)__popcll(m);
            __syncthreads();
            if (valid) {
                uint32_t pos = s_base[d] + rank;
                for (int w = 0; w < wave; ++w) pos += wcnt[w][d];
                if ((int64_t)pos < n) {
                    kout[pos] = k[it];
                    vout[pos] = val[it];
                }
            }
            __syncthreads();
            uint32_t add = 0;
            for (int w = 0; w < kSortThreads / 64; ++w) {
                add += wcnt[w][tid];
                wcnt[w][tid] = 0;
            }
            s_base[tid] += add;
            __syncthreads();
        }
    }
}

// Counts of the cells from the sorted keys, after the digit passes: one atomic per
// run of equal keys inside a wave.
__global__ void __launch_bounds__(256) k_run_count(const uint32_t *__restrict__ sk, int64_t n, uint32_t *__restrict__ cnt,
                                                   const int32_t *__restrict__ skip)
{
    if (skip && skip[1]) return;
    const int lane = threadIdx.x & 63;
    for (int64_t q0 = (int64_t)blockIdx.x * 256; q0 < n; q0 += (int64_t)gridDim.x * 256) {
        const int64_t q = q0 + threadIdx.x;
        const bool valid = q < n;
        const uint32_t k = valid ? sk[q] : 0u;
        const uint32_t before = __shfl_up(k, 1);
        const uint64_t starts = __ballot(valid && (lane == 0 || before != k)) | (~__ballot(valid));
        if (valid && ((starts >> lane) & 1ull)) atomicAdd(&cnt[k], (uint32_t)run_length(starts));
    }
}

// One workgroup sorts the distinct indices a[b..e) (all below n) into
// out[b..e) by 8-bit digits, through t; a and t are overwritten.
__device__ inline void sort_long_cell(int32_t *a, int32_t *t, int32_t *__restrict__ out, int64_t b, int64_t e,
                                      int64_t n, uint32_t *s_base, uint32_t (*wcnt)[256], uint32_t *lds)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint64_t lt = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int passes = 1;
    while (passes < 4 && ((n - 1) >> (8 * passes)) != 0) ++passes;
    for (int p = 0; p < passes; ++p) {
        const int32_t *in = (p & 1) ? t : a;
        int32_t *dst = p == passes - 1 ? out : ((p & 1) ? a : t);
        const int shift = 8 * p;
        s_base[tid] = 0;
        for (int w = 0; w < 4; ++w) wcnt[w][tid] = 0;
        __syncthreads();
        for (int64_t i = b + tid; i < e; i += 256) atomicAdd(&s_base[((uint32_t)in[i] >> shift) & 255u], 1u);
        __syncthreads();
        const uint32_t g = s_base[tid];
        uint32_t total;
        const uint32_t ex = block_scan_inclusive(g, lds, &total) - g;
        s_base[tid] = ex;
        __syncthreads();
        for (int64_t i0 = b; i0 < e; i0 += 256) {
            const int64_t i = i0 + tid;
            const bool valid = i < e;
            const int32_t v = valid ? in[i] : 0;
            const uint32_t d = ((uint32_t)v >> shift) & 255u;
            const uint64_t m = digit_mask(d, valid);
            const uint32_t rank = (uint32_t)__popcll(m & lt);
            if (valid && rank == 0) wcnt[wave][d] = (uint32_t)__popcll(m);
            __syncthreads();
            if (valid) {
                uint32_t pos = s_base[d] + rank;
                for (int w = 0; w < wave; ++w) pos += wcnt[w][d];
                dst[b + pos] = v;
            }
            __syncthreads();
            uint32_t add = 0;
            for (int w = 0; w < 4; ++w) {
                add += wcnt[w][tid];
                wcnt[w][tid] = 0;
            }
            s_base[tid] += add;
            __syncthreads();
        }
    }
}

// The granules of every cell in input order: a granule's place is the number
// of smaller indices in its cell (a cell's reads hit L1).  A cell of more than
// kLongCell granules, where that would grow with the square of its size, is
// sorted by digits by the workgroup that holds its first place.
constexpr int kLongCell = 256;

__global__ void __launch_bounds__(256) k_cell_order(int64_t n, const uint32_t *__restrict__ skeys,
                                                    const uint32_t *__restrict__ begin,
                                                    const uint32_t *__restrict__ end, int32_t *tmp, int32_t *tmp2,
                                                    int32_t *__restrict__ order, const int32_t *__restrict__ ctl,
                                                    int keep, uint32_t *__restrict__ cnt, int64_t K)
{
    if (keep && ctl[2]) return;
    if (cnt)  // the counts, for the next sort
        for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < K; k += (int64_t)gridDim.x * 256) cnt[k] = 0u;
    if (ctl && ctl[1]) return;
    __shared__ uint32_t s_base[256], wcnt[4][256], lds[4];
    __shared__ int64_t s_long[2];
    for (int64_t p0 = (int64_t)blockIdx.x * 256; p0 < n; p0 += (int64_t)gridDim.x * 256) {
        if (threadIdx.x == 0) s_long[1] = 0;
        __syncthreads();
        const int64_t p = p0 + threadIdx.x;
        if (p < n) {
            const uint32_t k = skeys[p];
            int64_t b = begin[k], e = end[k];
            e = e < n ? e : n;
            if (e - b <= kLongCell) {
                const int32_t v = tmp[p];
                int rank = 0;
                for (int64_t j = b; j < e; ++j) rank += tmp[j] < v ? 1 : 0;
                order[b + rank] = v;
            } else if (p == b) {  // at most one such cell begins in 256 places
                s_long[0] = b;
                s_long[1] = e;
            }
        }
        __syncthreads();
        if (s_long[1]) sort_long_cell(tmp, tmp2, order, s_long[0], s_long[1], n, s_base, wcnt, lds);
        __syncthreads();
    }
}

// The last pass of a rollout step's sort: the order of k_cell_order, and with it
// the state in sorted order (xv: x then v in input order), the grid sums fx
// (len int64) cleared, and each workgroup's largest granule fraction in part.
// REV (the reverse step): also the adjoint of the state in sorted order, moved
// through the integration: v^{n+1} feeds x^{n+1}, so its adjoint, which is also
// that of v^n through the identity term, is g_v + dt g_x, and the adjoint of
// the force is dt / m of it.  ORDERED: the digit passes have left the order.
template <bool REV, bool ORDERED>
__global__ void __launch_bounds__(256) k_rollout_order(DevParams P, int64_t n, const uint32_t *__restrict__ skeys,
                                                       const uint32_t *__restrict__ begin,
                                                       const uint32_t *__restrict__ end, int32_t *tmp, int32_t *tmp2,
                                                       int32_t *__restrict__ order, uint32_t *__restrict__ cnt, int64_t K,
                                                       const double *__restrict__ xv, const double *__restrict__ r,
                                                       double *__restrict__ xvs, double *__restrict__ rs,
                                                       int64_t *__restrict__ fx, int64_t len, double *__restrict__ part,
                                                       const double *__restrict__ gxv, double *__restrict__ gs,
                                                       double *__restrict__ gF, unsigned long long *__restrict__ gmax)
{
    __shared__ uint32_t s_base[256], wcnt[4][256], lds[4];
    __shared__ int64_t s_long[2];
    __shared__ double s_m[4];
    if (cnt)  // the counts, for the next sort
        for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < K; k += (int64_t)gridDim.x * 256) cnt[k] = 0u;
    for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < len; k += (int64_t)gridDim.x * 256) fx[k] = 0;
    if (REV && blockIdx.x == 0 && threadIdx.x == 0) *gmax = 0ull;
    double m = 0.0;
    auto take = [&](int64_t q, int64_t i) {  // granule i at sorted position q
        double s[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) s[c] = xv[c * n + i];
        const double ri = r[i];
        if (REV) {
            const double w = P.dt / mass_of(P, ri);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double gx = gxv[a * n + i];
                const double t = gxv[(3 + a) * n + i] + P.dt * gx;
                gs[a * n + q] = gx;
                gs[(3 + a) * n + q] = t;
                gF[a * n + q] = w * t;
            }
        }
#pragma unroll
        for (int c = 0; c < 6; ++c) xvs[c * n + q] = s[c];
        rs[q] = ri;
        m = fmax(m, volume_of(ri) * P.inv_vcell);
    };
    if constexpr (ORDERED)
        for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (int64_t)gridDim.x * 256) take(q, order[q]);
    for (int64_t p0 = (int64_t)blockIdx.x * 256; !ORDERED && p0 < n; p0 += (int64_t)gridDim.x * 256) {
        if (threadIdx.x == 0) s_long[1] = 0;
        __syncthreads();
        const int64_t p = p0 + threadIdx.x;
        if (p < n) {
            const uint32_t k = skeys[p];
            int64_t b = begin[k], e = end[k];
            e = e < n ? e : n;
            if (e - b <= kLongCell) {
                const int32_t v = tmp[p];
                int rank = 0;
                for (int64_t j = b; j < e; ++j) rank += tmp[j] < v ? 1 : 0;
                order[b + rank] = v;
                take(b + rank, v);
            } else if (p == b) {  // at most one such cell begins in 256 places
                s_long[0] = b;
                s_long[1] = e;
            }
        }
        __syncthreads();
        if (s_long[1]) {
            sort_long_cell(tmp, tmp2, order, s_long[0], s_long[1], n, s_base, wcnt, lds);
            __syncthreads();
            for (int64_t q = s_long[0] + threadIdx.x; q < s_long[1]; q += 256) take(q, order[q]);
        }
        __syncthreads();
    }
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(s_m[0], s_m[1]), fmax(s_m[2], s_m[3]));
}

__global__ void __launch_bounds__(256) k_reorder(int64_t n, const int32_t *__restrict__ order,
                                                 const double *__restrict__ x, const double *__restrict__ v,
                                                 const double *__restrict__ r, const int32_t *__restrict__ id,
                                                 double *__restrict__ xo, double *__restrict__ vo,
                                                 double *__restrict__ ro, int32_t *__restrict__ ido)
{
    int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    int64_t i = order[q];
    if ((uint64_t)i >= (uint64_t)n) return;  // not a permutation of [0, n): position q left untouched
    for (int a = 0; a < 3; ++a) {
        xo[a * n + q] = x[a * n + i];
        vo[a * n + q] = v[a * n + i];
    }
    ro[q] = r[i];
    if (ido) ido[q] = id[i];
}

// ---- incremental path: few keys changed since the last sort -------------
//
// The previous sorted keys pk are non-decreasing by position, so the
// granules whose key still equals pk at their position (U) are in sorted
// order already, whatever state they come from; the others (C, at most
// kChgCap) are sorted here.  The stable sort by (key, position) is then the
// merge of U and C: an element's place is the number of U elements before
// it plus the number of C elements before it.  For u in U at position i
// that is (i - #C positions below i) + #C pairs below (key, i); for c in C
// it is its rank in C plus #U pairs below (k_c, i_c) = L - #C positions
// below L, with L the number of positions i with (pk[i], i) < (k_c, i_c).

// One workgroup: decides the path, sorts C by (key, position) and by
// position (bitonic, in LDS), and places the C elements.  With nl it also
// decides whether the neighbour list must be rebuilt this step (nl[0]):
// when force is set, when any key changed (the sorted order may change), or
// when the largest squared displacement since the build (the maximum of the
// nd per-workgroup maxima dpart of the key kernel) reaches thr2.
__global__ void __launch_bounds__(1024) k_chg_sort(int64_t n, const uint32_t *__restrict__ pk,
                                                   const uint64_t *__restrict__ chg, int32_t *__restrict__ ctl,
                                                   uint64_t *__restrict__ chg_s, uint32_t *__restrict__ chg_p,
                                                   uint32_t *__restrict__ skeys, int32_t *__restrict__ order,
                                                   uint32_t *__restrict__ nl, int force, float thr2,
                                                   const float *__restrict__ dpart, int64_t nd)
{
    __shared__ uint64_t sk[kChgCap];
    __shared__ uint32_t sp[kChgCap];
    __shared__ float s_dm[1024 / 64];
    const int tid = threadIdx.x;
    const int m = ctl[0];
    const bool incremental = m <= kChgCap;
    float dm = 0.0f;
    if (dpart)
        for (int64_t i = tid; i < nd; i += 1024) dm = fmaxf(dm, dpart[i]);
    for (int off = 32; off > 0; off >>= 1) dm = fmaxf(dm, __shfl_xor(dm, off));
    if ((tid & 63) == 0) s_dm[tid >> 6] = dm;
    __syncthreads();  // every thread has read ctl[0] before thread 0 writes ctl[1]
    if (tid == 0) {
        ctl[1] = incremental ? 1 : 0;
        ctl[2] = m == 0 ? 1 : 0;  // no key changed: the last sort's order, ranges and bricks hold
    }
    if (tid == 0 && nl) {
        float d2 = 0.0f;
        for (int w = 0; w < 1024 / 64; ++w) d2 = fmaxf(d2, s_dm[w]);
        nl[0] = (force || m != 0 || !(d2 < thr2)) ? 1u : 0u;
    }
    if (!incremental || m == 0) return;
    int N = 2;
    while (N < m) N <<= 1;
    for (int i = tid; i < N; i += 1024) {
        const uint64_t e = i < m ? chg[i] : ~0ull;
        sk[i] = e;
        sp[i] = i < m ? (uint32_t)(e & 0xffffffffu) : 0xffffffffu;
    }
    __syncthreads();
    for (int k = 2; k <= N; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = tid; i < N; i += 1024) {
                const int l = i ^ j;
                if (l > i) {
                    const bool up = (i & k) == 0;
                    const uint64_t a = sk[i], b = sk[l];
                    if ((a > b) == up) {
                        sk[i] = b;
                        sk[l] = a;
                    }
                    const uint32_t c = sp[i], d = sp[l];
                    if ((c > d) == up) {
                        sp[i] = d;
                        sp[l] = c;
                    }
                }
            }
            __syncthreads();
        }
    for (int r = tid; r < m; r += 1024) {
        chg_s[r] = sk[r];
        chg_p[r] = sp[r];
        const uint32_t kc = (uint32_t)(sk[r] >> 32), ic = (uint32_t)(sk[r] & 0xffffffffu);
        int64_t lo = 0, hi = n;  // L: positions i with (pk[i], i) < (kc, ic)
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            const uint32_t pm = pk[mid];
            if (pm < kc || (pm == kc && mid < (int64_t)ic)) lo = mid + 1; else hi = mid;
        }
        const int64_t place = r + lo - lower_bound_u32(sp, m, (uint32_t)lo);
        order[place] = (int32_t)ic;
        skeys[place] = kc;
    }
}

// ---- occupied bricks, in brick order (the schedule of the brick kernels) ----

__device__ inline bool brick_occupied(int64_t b, const int32_t *__restrict__ cb, const int32_t *__restrict__ ce)
{
    return ce[b * kBrickCells + kBrickCells - 1] > cb[b * kBrickCells];
}

__global__ void __launch_bounds__(256) k_brick_count(int64_t nbricks, int64_t per_block, const int32_t *__restrict__ cb,
                                                     const int32_t *__restrict__ ce, uint32_t *__restrict__ sums)
{
    __shared__ uint32_t lds[4];
    const int64_t lo = (int64_t)blockIdx.x * per_block;
    const int64_t hi = lo + per_block < nbricks ? lo + per_block : nbricks;
    uint32_t c = 0;
    for (int64_t b = lo + threadIdx.x; b < hi; b += 256) c += brick_occupied(b, cb, ce) ? 1u : 0u;
    c = block_reduce_sum(c, lds);
    if (threadIdx.x == 0) sums[blockIdx.x] = c;
}

// The whole list in one workgroup, for few bricks.
constexpr int64_t kBricksOneGroup = 2048;

__global__ void __launch_bounds__(kScanThreads) k_brick_list(int nbricks, const int32_t *__restrict__ cb,
                                                             const int32_t *__restrict__ ce,
                                                             int32_t *__restrict__ list, int32_t *__restrict__ count,
                                                             int32_t *__restrict__ slot_of, int32_t n)
{
    constexpr int kRounds = (int)(kBricksOneGroup / kScanThreads);
    __shared__ uint32_t lds[kScanThreads / 64];
    // thread t takes kRounds consecutive bricks (all loads in flight together)
    const int b0 = (int)threadIdx.x * kRounds;
    int32_t lo[kRounds], hi[kRounds];
#pragma unroll
    for (int u = 0; u < kRounds; ++u) {
        const int b = b0 + u < nbricks ? b0 + u : nbricks - 1;
        lo[u] = cb[(int64_t)b * kBrickCells];
        hi[u] = ce[(int64_t)b * kBrickCells + kBrickCells - 1];
    }
    uint32_t f = 0;
#pragma unroll
    for (int u = 0; u < kRounds; ++u) f += b0 + u < nbricks && hi[u] > lo[u] ? 1u : 0u;
    uint32_t total;
    uint32_t at = block_scan_inclusive(f, lds, &total) - f;
#pragma unroll
    for (int u = 0; u < kRounds; ++u) {
        if (b0 + u >= nbricks) break;
        const bool occ = hi[u] > lo[u];
        slot_of[b0 + u] = occ ? (int32_t)at : -1;
        if (occ) list[at++] = b0 + u;
    }
    if (threadIdx.x == 0) put_count(count, (int32_t)total, n, false);
}

// Each workgroup sums the counts before its own (at most kScanThreads words).
__global__ void __launch_bounds__(256) k_brick_scatter(int64_t nbricks, int64_t per_block,
                                                       const int32_t *__restrict__ cb, const int32_t *__restrict__ ce,
                                                       const uint32_t *__restrict__ sums, int32_t *__restrict__ list,
                                                       int32_t *__restrict__ count, int32_t *__restrict__ slot_of,
                                                       int32_t n)
{
    __shared__ uint32_t lds[4];
    __shared__ uint32_t s_base;
    const int64_t lo = (int64_t)blockIdx.x * per_block;
    const int64_t hi = lo + per_block < nbricks ? lo + per_block : nbricks;
    uint32_t base = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += 256) base += sums[t];
    base = block_reduce_sum(base, lds);
    if (threadIdx.x == 0) s_base = base;
    __syncthreads();
    base = s_base;
    for (int64_t b0 = lo; b0 < hi; b0 += 256) {  // same trip count for the whole workgroup
        const int64_t b = b0 + threadIdx.x;
        const uint32_t f = b < hi && brick_occupied(b, cb, ce) ? 1u : 0u;
        uint32_t total;
        const uint32_t inc = block_scan_inclusive(f, lds, &total);
        if (f) list[base + inc - 1] = (int32_t)b;
        if (b < hi) slot_of[b] = f ? (int32_t)(base + inc - 1) : -1;
        base += total;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) put_count(count, (int32_t)base, n, false);
}

// Samples of a bed for its record, one workgroup.
//
// How full the groups are (groups; see fill_mode), from kGroupSample groups spread
// over the box, each at a place of its own in its share so that no bed's period
// falls in with theirs.  And how many of kDenseSample sorted granules lie in cells
// of more than limit (skeys given; see sort_by_digits), as a share of n: all, if one
// lies in a cell of more than longest (so many that a sample meets it).
__global__ void __launch_bounds__(1024) k_bed_sample(int32_t nbx, int32_t nby, int32_t nbz, int64_t n, int groups_too,
                                                     uint32_t limit, uint32_t longest,
                                                     const int32_t *__restrict__ slot_of,
                                                     const uint32_t *__restrict__ skeys,
                                                     const uint32_t *__restrict__ begin, const uint32_t *__restrict__ end,
                                                     int32_t *__restrict__ count)
{
    __shared__ uint32_t lds[1024 / 64];
    if (skeys) {
        uint32_t dense = 0;
        bool one = false;
#pragma unroll
        for (int u = 0; u < kDenseSample / 1024; ++u) {
            const int64_t p = (threadIdx.x + u * 1024) * n / kDenseSample;
            const uint32_t k = skeys[p];
            const uint32_t len = end[k] - begin[k];
            dense += len > limit ? 1u : 0u;
            one |= len > longest;
        }
        one = __syncthreads_or(one);
        dense = block_reduce_sum(dense, lds);
        if (threadIdx.x == 0) count[5] = one ? (int32_t)n : (int32_t)((int64_t)dense * n / kDenseSample);
    }
    if (!groups_too) return;
    const uint32_t ngx = (uint32_t)(nbx + kGroup - 1) / kGroup, ngy = (uint32_t)(nby + kGroup - 1) / kGroup;
    const uint32_t groups = ngx * ngy * ((uint32_t)(nbz + kGroup - 1) / kGroup);  // below 2^31, as the bricks are
    uint32_t held = 0, occ = 0;
#pragma unroll
    for (int u = 0; u < kGroupSample / 1024; ++u) {
        const uint32_t t = threadIdx.x + u * 1024;
        const uint32_t lo = (uint32_t)((uint64_t)t * groups / kGroupSample);
        const uint32_t share = (uint32_t)((uint64_t)(t + 1) * groups / kGroupSample) - lo;
        const uint32_t g = lo + (share > 1 ? (t * 2654435761u >> 8) % share : 0u);
        const uint32_t gyz = g / ngx, gz = gyz / ngy;
        const int32_t bx = (int32_t)(g - gyz * ngx) * kGroup, by = (int32_t)(gyz - gz * ngy) * kGroup;
        const int32_t bz = (int32_t)gz * kGroup;
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kGroup * kGroup * kGroup; ++w) {
            const int32_t x = bx + w % kGroup, y = by + w / kGroup % kGroup, z = bz + w / (kGroup * kGroup);
            if (share != 0u && x < nbx && y < nby && z < nbz)
                c += slot_of[((int64_t)z * nby + y) * nbx + x] >= 0 ? 1u : 0u;
        }
        held += c != 0u ? 1u : 0u;
        occ += c;
    }
    held = block_reduce_sum(held, lds);
    occ = block_reduce_sum(occ, lds);
    if (threadIdx.x == 0) {
        count[2] = (int32_t)held;
        count[3] = (int32_t)occ;
    }
}

}  // namespace

namespace {

constexpr unsigned kLoopGrid = 2048;  // workgroups of 256 that the chip holds at once

// A sort's keys and ranges, for its record.
struct Sorted {
    const uint32_t *skeys, *begin, *end;
    int64_t limit;
    bool asks;  // the next sort's form depends on whether this one's input was shuffled
};

// Every 16th list, and the first of another number of granules, leaves its record
// in pinned host memory (see brick_fill).  So do the first sort among them and,
// where the next asks for what changed, the second (the first that can be compared).
// Samples are taken of those, and of every 64th list (groups) and sort (cells).
hipError_t brick_count_copy(const DevParams &P, BrickList &B, int64_t n, hipStream_t s, const Sorted &S = Sorted{})
{
    hipError_t e = hipGetLastError();
    if (n <= 0 || !B.seen) return e;
    if (B.seen_n != n) B.calls = B.sorts = 0;
    B.seen_n = n;
    const bool sort = S.skeys != nullptr;
    const unsigned call = B.calls++, nth = sort ? B.sorts++ : 0;
    const bool fresh = call == 0 || (sort && (nth == 0 || (nth == 1 && S.asks)));
    const bool cells = sort && n >= kDenseSorts && (fresh || (nth & 63u) == 0u);
    if (!fresh && !cells && (call & 15u) != 0u) return e;
    // (groups: where the bed may be run by them, as far as is known)
    const bool groups = n >= kWaveBricks * kBrickCells && B.nbricks >= kGroupBricks && brick_fill(P, n, B).avg <= kWaveFill;
    const bool sampled = groups && (fresh || (call & 63u) == 0u);
    if (sampled || cells) {
        k_bed_sample<<<1, 1024, 0, s>>>(P.nb[0], P.nb[1], P.nb[2], n, sampled ? 1 : 0,
                                        (uint32_t)(S.limit ? S.limit : sort_limit(n, false)), (uint32_t)sort_long(n), B.slot_of,
                                        cells ? S.skeys : nullptr, S.begin, S.end, B.count);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(B.seen, B.count, sizeof(BrickSeen), hipMemcpyDeviceToHost, s);
    return e;
}

int64_t scan_chunk(int64_t len)
{
    const int64_t chunk = (len + kScanThreads - 1) / kScanThreads, unit = 4 * kScanThreads;
    return (chunk + unit - 1) / unit * unit;
}

}  // namespace

namespace {

// The digit passes of a sort: skeys and order from key.
void digit_passes(int64_t n, const uint32_t *key, uint32_t *skeys, int32_t *order, SortScratch &S, const int32_t *skip,
                  hipStream_t s)
{
    const int64_t tiles = sort_tiles(n);
    const unsigned tg = (unsigned)(tiles < kDigitGrid ? tiles : kDigitGrid);
    const uint32_t *kin = key;
    const int32_t *vin = nullptr;
    for (int pass = 0; pass < S.passes; ++pass) {
        const bool last = pass == S.passes - 1;
        uint32_t *kout = ((S.passes - 1 - pass) & 1) ? S.slot : skeys;  // the last into skeys
        int32_t *vout = last ? order : ((pass & 1) ? S.tmp2 : S.tmp);
        if (sort_items(n) == 1)
            k_digit_count<1><<<tg, kSortThreads, 0, s>>>(kin, n, pass, tiles, S.tcnt, skip);
        else
            k_digit_count<kSortItems><<<tg, kSortThreads, 0, s>>>(kin, n, pass, tiles, S.tcnt, skip);
        k_digit_scan<<<256, kSortThreads, 0, s>>>(S.tcnt, tiles, S.rowtot, skip);
        if (sort_items(n) == 1)
            k_digit_scatter<1><<<tg, kSortThreads, 0, s>>>(kin, vin, kout, vout, n, pass, tiles, S.tcnt, S.rowtot, skip);
        else
            k_digit_scatter<kSortItems>
                <<<tg, kSortThreads, 0, s>>>(kin, vin, kout, vout, n, pass, tiles, S.tcnt, S.rowtot, skip);
        kin = kout;
        vin = vout;
    }
}

}  // namespace

hipError_t launch_sort_cells(const DevParams &P, int64_t n, const double *x, uint32_t *key, int32_t *order,
                             int32_t *cell_begin, int32_t *cell_end, int64_t K, SortScratch &S, BrickList &B,
                             int64_t *err, hipStream_t s, const NbrList *nl, int force, int keep_ranges)
{
    B.use = B.list;
    B.use_count = B.count;
    uint32_t *cnt = S.cnt;  // all zero between sorts
    uint32_t *begin = reinterpret_cast<uint32_t *>(cell_begin), *end = reinterpret_cast<uint32_t *>(cell_end);
    // previous sorted keys: usable when the last sort had the same n
    const bool same_n = n > 0 && S.last_n == n;
    const int keep = keep_ranges && same_n ? 1 : 0;
    // a stepping call continues a sorted state; what a stage call sorts, the
    // record of its last sorts says
    const volatile BrickSeen *seen = B.seen;
    const bool shuffled = !same_n || (!nl && !(seen && seen->n == n && 2 * (int64_t)seen->changed <= n));
    const int64_t limit = sort_limit(n, shuffled);
    const bool digits = n > 0 && sort_by_digits(n, K, B, limit);
    const bool small = n <= kSmallSort && !digits;
    // a small sort compares with the previous keys only where an unchanged
    // state saves the rest of it or the neighbour list
    const bool inc = same_n && (!small || keep || (nl && !force));
    const uint32_t *pk = inc ? S.skeys[S.cur] : nullptr;
    uint32_t *skeys = S.skeys[S.cur ^ 1];
    int32_t *ctl = inc ? S.ctl : nullptr;
    // the displacement since the list's build is measured when the list may
    // be kept (its build had this sorted order: the caller checked that)
    const bool measure = nl && inc && !force && nl->thr2 > 0.0f;
    const unsigned g = grid_for(n, 256);
    // the passes that may have nothing to do loop over a resident grid: an idle
    // launch of 65,536 workgroups took 15 us
    const unsigned gl = g < kLoopGrid ? g : kLoopGrid;
    uint32_t *nctl = nl ? nl->ctl : nullptr;
    const float thr2 = nl ? nl->thr2 : 0.0f;
    float *dpart = measure ? nl->dpart : nullptr;
    if (n > 0) {
        k_cell_keys<<<g, 256, 0, s>>>(P, n, x, key, err, pk, small ? nullptr : S.chg, S.ctl,
                                      measure ? nl->xref : nullptr, dpart, order, skeys);
        if (inc && !small)
            k_chg_sort<<<1, 1024, 0, s>>>(n, pk, S.chg, S.ctl, S.chg_s, S.chg_p, skeys, order, nctl, measure ? 0 : 1,
                                          thr2, dpart, (int64_t)g);
        if (inc || !digits)
            k_cell_count<<<gl, 256, 0, s>>>(key, n, cnt, S.slot, pk, S.chg_s, S.chg_p, skeys, order, ctl,
                                            digits ? 2 : (inc && small ? 1 : 0), keep, nctl, measure ? 0 : 1, thr2,
                                            dpart, (int64_t)g);
        if (digits) {
            digit_passes(n, key, skeys, order, S, ctl, s);
            k_run_count<<<gl, 256, 0, s>>>(skeys, n, cnt, ctl);
        }
    }
    // cell ranges and bricks: kept when the caller's tables hold the last
    // sort's ranges and no key changed (decided on the device)
    // (tables of one pass: chunks of 4,096 cells, so that 32 workgroups share them)
    const bool direct = n > 0 && K <= kDirectScan && !digits;
    const int64_t chunk = direct ? 4 * kScanThreads : scan_chunk(K);
    const int nb = (int)((K + chunk - 1) / chunk);
    if (!direct)
        k_scan_reduce<<<nb, kScanThreads, 0, s>>>(cnt, K, chunk, S.sums, S.sums + kScanThreads,
                                                  keep ? S.ctl : nullptr);
    k_scan_down_ranges<<<nb, kScanThreads, 0, s>>>(cnt, begin, end, K, chunk, direct ? nullptr : S.sums,
                                                   S.sums + kScanThreads, S.ctl, keep, B.list, B.count, B.slot_of,
                                                   (int32_t)n, inc ? 1 : 0);
    if (n > 0 && !digits) {
        k_cell_place<<<gl, 256, 0, s>>>(key, n, begin, S.slot, S.tmp, skeys, ctl, keep);
        k_cell_order<<<gl, 256, 0, s>>>(n, skeys, begin, end, S.tmp, S.tmp2, order, ctl, keep, direct ? cnt : nullptr,
                                        K);
    }
    S.cur ^= 1;  // this sort's keys are the previous keys of the next
    S.last_n = n;
    return brick_count_copy(P, B, n, s, Sorted{skeys, begin, end, limit, !nl && n > kSmallSort});
}

hipError_t launch_rollout_sort(const DevParams &P, int64_t n, const double *xv, const double *r, uint32_t *key,
                               int32_t *order, int32_t *cell_begin, int32_t *cell_end, int64_t K, SortScratch &S,
                               BrickList &B, int64_t *err, double *xvs, double *rs, int64_t *fx, int64_t len,
                               double *part, int *nb, const double *gxv, double *gs, double *gF,
                               unsigned long long *gmax, hipStream_t s)
{
    B.use = B.list;
    B.use_count = B.count;
    uint32_t *begin = reinterpret_cast<uint32_t *>(cell_begin), *end = reinterpret_cast<uint32_t *>(cell_end);
    uint32_t *skeys = S.skeys[S.cur ^ 1];
    const int64_t limit = sort_limit(n, true, true);  // input order
    const bool digits = sort_by_digits(n, K, B, limit);
    const unsigned g = grid_for(n, 256), gl = g < kLoopGrid ? g : kLoopGrid, go = g < 1024u ? g : 1024u;
    k_cell_keys<<<g, 256, 0, s>>>(P, n, xv, key, err, nullptr, nullptr, S.ctl, nullptr, nullptr, order, skeys);
    if (digits) {
        digit_passes(n, key, skeys, order, S, nullptr, s);
        k_run_count<<<gl, 256, 0, s>>>(skeys, n, S.cnt, nullptr);
    } else {
        k_cell_count<<<gl, 256, 0, s>>>(key, n, S.cnt, S.slot, nullptr, S.chg_s, S.chg_p, skeys, order, nullptr, 0, 0,
                                        nullptr, 1, 0.0f, nullptr, 0);
    }
    const bool direct = K <= kDirectScan && !digits;
    const int64_t chunk = direct ? 4 * kScanThreads : scan_chunk(K);
    const int nc = (int)((K + chunk - 1) / chunk);
    if (!direct)
        k_scan_reduce<<<nc, kScanThreads, 0, s>>>(S.cnt, K, chunk, S.sums, S.sums + kScanThreads, nullptr);
    k_scan_down_ranges<<<nc, kScanThreads, 0, s>>>(S.cnt, begin, end, K, chunk, direct ? nullptr : S.sums,
                                                   S.sums + kScanThreads, S.ctl, 0, B.list, B.count, B.slot_of, (int32_t)n,
                                                   0);
    if (!digits) k_cell_place<<<gl, 256, 0, s>>>(key, n, begin, S.slot, S.tmp, skeys, nullptr, 0);
    uint32_t *cnt = direct ? S.cnt : nullptr;
#define GIC_ROLLOUT_ORDER(REV, ORDERED)                                                                                \
    k_rollout_order<REV, ORDERED><<<go, 256, 0, s>>>(P, n, skeys, begin, end, S.tmp, S.tmp2, order, cnt, K, xv, r,     \
                                                     xvs, rs, fx, len, part, gxv, gs, gF, gmax)
    if (gxv) {
        if (digits)
            GIC_ROLLOUT_ORDER(true, true);
        else
            GIC_ROLLOUT_ORDER(true, false);
    } else {
        if (digits)
            GIC_ROLLOUT_ORDER(false, true);
        else
            GIC_ROLLOUT_ORDER(false, false);
    }
#undef GIC_ROLLOUT_ORDER
    *nb = (int)go;
    S.cur ^= 1;
    S.last_n = n;
    return brick_count_copy(P, B, n, s, Sorted{skeys, begin, end, limit, false});
}

hipError_t launch_brick_list(const DevParams &P, const int32_t *cb, const int32_t *ce, BrickList &B, int64_t n,
                             hipStream_t s)
{
    B.use = B.list;
    B.use_count = B.count;
    const int64_t nb = B.nbricks;
    if (nb <= 0) return hipSuccess;
    if (nb <= kBricksOneGroup) {
        k_brick_list<<<1, kScanThreads, 0, s>>>((int)nb, cb, ce, B.list, B.count, B.slot_of, (int32_t)n);
        return brick_count_copy(P, B, n, s);
    }
    int64_t per = 1024;
    while ((nb + per - 1) / per > kScanThreads) per *= 2;
    const int blocks = (int)((nb + per - 1) / per);
    k_brick_count<<<blocks, 256, 0, s>>>(nb, per, cb, ce, B.sums);
    k_brick_scatter<<<blocks, 256, 0, s>>>(nb, per, cb, ce, B.sums, B.list, B.count, B.slot_of, (int32_t)n);
    return brick_count_copy(P, B, n, s);
}

void box_list(int64_t n, int32_t *out)
{
    const int64_t per = (n + kXcds - 1) / kXcds;
    int64_t at[kXcds];  // next free entry of each eighth
    for (int x = 0; x < kXcds; ++x) at[x] = x * per;
    auto room = [&](int x) { return at[x] < (x + 1) * per && at[x] < n; };
    int x = 0;
    for (int64_t b = 0; b < n; ++b) {
        if (b % 16 == 0) x = (int)(b / 16 % kXcds);
        while (!room(x)) x = (x + 1) % kXcds;  // the eighths hold n entries in all
        out[at[x]++] = (int32_t)b;
    }
    out[n] = (int32_t)n;
}

hipError_t launch_reorder(int64_t n, const int32_t *order, const double *x, const double *v, const double *r,
                          const int32_t *id, double *xo, double *vo, double *ro, int32_t *ido, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_reorder<<<grid_for(n, 256), 256, 0, s>>>(n, order, x, v, r, ido ? id : nullptr, xo, vo, ro, ido);
    return hipGetLastError();
}

}  // namespace gic
