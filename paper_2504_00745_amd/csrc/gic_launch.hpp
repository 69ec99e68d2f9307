// Host-side launchers of the gfx950 kernels (one translation unit per stage
// family); the C ABI in gic_api.hip validates arguments and calls these.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gic_device.hpp"

namespace gic {

// Granules whose key changed since the last sort that the incremental path
// takes (more: everything is counted again).
constexpr int kChgCap = 4096;

// Sort scratch owned by a context.
struct SortScratch {
    uint32_t *skeys[2];  // sorted keys; skeys[cur] holds those of the last sort
    int cur;
    int64_t last_n;      // granules of the last sort, -1 before the first
    uint32_t *slot;      // [n] place of each granule in its cell, in order of arrival
    int32_t *tmp, *tmp2; // [n] granules by cell, in order of arrival; second array of long cells
                         // (digit passes: the values' buffers; slot and the sorted keys are the keys')
    int passes;          // 8-bit digits of the keys
    uint32_t *sums;      // [2 x 1024] granules and occupied bricks of the scan's chunks
    uint32_t *rowtot;    // [256] keys with each digit in a digit pass (after sums, in its allocation)
    uint32_t *tcnt;      // [256][sort_tiles_max] digit counts, then output offsets, of each tile in a digit
                         // pass (in the array of a deposit's escapes: no sort runs inside a deposit)
    uint32_t *cnt;       // [K] granules per cell; zero between sorts
    uint64_t *chg;       // [kChgCap] changed granules as (key << 32 | position), in arrival order
    uint64_t *chg_s;     // [kChgCap] the same sorted
    uint32_t *chg_p;     // [kChgCap] their positions sorted
    int32_t *ctl;        // [4] changed count (zero between sorts), path of this sort (1 = incremental),
                         // no key changed (1: order, ranges and bricks of the last sort hold), spare
};

// What the host learns of a brick list, without waiting: its occupied bricks and
// the granules it was built for (a record in flight when the next bed's list is
// built names its own bed), and, for beds large enough to be run by groups, the
// groups of a sample that hold granules and their occupied bricks (0: none taken).
// Of the last sort: the granules whose key had changed since the one before (all,
// where they were not compared); of the last sampled, those in cells larger than
// its sort_limit (all, if one lies in a cell of more than sort_long; -1: none sampled).
struct BrickSeen {
    int32_t count, n;
    int32_t groups, bricks;
    int32_t changed, dense;
};
// Groups and granules of the samples; fixed numbers, so that taking them costs the
// same in any box.  Sorts of fewer than kDenseSorts granules are not sampled.
constexpr int kGroupSample = 4096, kDenseSample = 4096;
constexpr int64_t kDenseSorts = 8192;

// Occupied bricks of a set of cell ranges, in brick order (see
// brick_of_block), built by launch_brick_list before the brick kernels.
struct BrickList {
    int32_t *list;     // [nbricks]
    int32_t *count;    // [6] their number, and the rest of a BrickSeen
    uint32_t *sums;    // [<= 1024] block totals
    int32_t *box;      // [nbricks + 1] every brick of the box and their number, or NULL (see box_list)
    const int32_t *use, *use_count;  // what the brick kernels run over: list and count, or the box
    int32_t *slot_of;  // [nbricks] position of each brick in list, -1 if empty
    int64_t nbricks;
    BrickSeen *seen;   // pinned host: a copy of an earlier list's count (see brick_fill)
    int64_t seen_n;    // granules of the last list
    unsigned calls, sorts;  // lists of seen_n granules in a row, and sorts among them
};

// Every brick of the box in the order of a brick list, runs of 16 neighbouring
// bricks to the XCDs' eighths in turn (a bed fills part of the box); host, n + 1
// int32, the last one n.
void box_list(int64_t n, int32_t *out);
// n: granules of the tables, or -1 when the caller does not know (no copy of
// the count to the host then).
hipError_t launch_brick_list(const DevParams &P, const int32_t *cb, const int32_t *ce, BrickList &B, int64_t n,
                             hipStream_t s);

// Persistent neighbour list of the contact stage (owned by a context): for
// every granule (sorted position q) the sorted positions of the granules
// closer than r_i + r_j + skin when the list was built, in the order of
// their cells (z, then y, then x) and of their positions inside a cell.  The
// contact kernel runs the exact test of Sec. 3.1 on the listed granules
// every step, so the list only has to hold every pair that can touch: it
// stays valid while the sorted order is unchanged and no granule has moved
// by skin / 2 since the build.
constexpr int kNbrCap = 16;  // partners listed per granule; more: the contact kernel searches the cells
struct NbrList {
    int32_t *nbr;   // [kNbrCap][n]: partner k of granule q at k * n + q
    int32_t *cnt;   // [n] partners found (> kNbrCap: not listed, searched)
    float *xref;    // [3][n] positions at the build
    uint32_t *ctl;  // [4] rebuild flag of this step, spare, builds, spare
    float *dpart;   // [n / 256] largest squared displacement since the build per key-kernel workgroup
    double skin;    // reach of the list beyond r_i + r_j [m]
    float thr2;     // squared displacement since the build that calls for a rebuild (< 0: every step)
};

// Up to this many keys a counting sort does not collect the changed ones:
// counting everything again is faster than merging them in.  Eight granules a
// cell, sorted but for none, 512, 4,000 and 5 % of them, counting against merging, us:
//   131,072: 19 to 25 in each case, and 22 to 29, 35, 84 and 27
//   262,144: 20 to 25, and 22 to 30, 38, 93 and 35
//   524,288: 27, and 24 to 32, 45, 111 and 53
//   1.05 million: 39, 53, 75 and 92 to 94, and 28 to 33, 53, 132 and 84
// Above it the changed keys are counted also where merging is no faster: their
// number says whether the next input is shuffled, on which the choice between
// counting and the digit passes depends there (see sort_limit).
constexpr int64_t kSmallSort = (int64_t)1 << 18;

// A sort counts, or passes over the keys' digits.  Counting places each granule
// with an atomic on its cell and a store, both at random where the input is
// shuffled, and puts a cell's granules in order at a cost that grows with the
// cell; the digit passes cost the same for any input.  sort_limit: the granules
// per cell from which the digits are faster, 0 for any; shuffled: most keys differ
// from those of the last sort at their place.  Counting against digits, us:
//   262,144, sorted 300 a cell 57 and 65; shuffled 96 60 and 65, 128 68 and 64
//   524,288, sorted 128 78 and 78; shuffled 8 89 and 99, 32 93 and 79
//   786,432, sorted 96 93 and 95, 128 101 and 96; shuffled 8 120 and 121, 32 126 and 100
//   4.2 million, sorted 64 354 and 353, 128 424 and 308; shuffled 1 580 and 477
//   16.8 million, sorted 32 1,228 and 1,344, 64 1,384 and 1,346; shuffled 1 2,493 and 1,947
// and 16 cells of 262,144 granules each, shuffled, 18,300 and 1,000.
// gathers: the counting sort's last pass gathers the state too (rollout; five
// steps of 592,704 granules 1,567 and 1,653, of 1.0 million 2,564 and 2,577, of 2.1
// million 5,715 and 5,632).
inline int64_t sort_limit(int64_t n, bool shuffled, bool gathers = false)
{
    if (n <= kSmallSort) return 160;
    if (shuffled) return n <= (gathers ? 4 : 2) * kSmallSort ? 32 : 0;
    return n <= 2 * kSmallSort ? 128 : (n <= 4 * kSmallSort ? 96 : 64);
}
// Whether a sort of n granules in K cells takes the digit passes, from the record
// of an earlier list of n granules or, before the first, from the mean of the box.
inline bool sort_by_digits(int64_t n, int64_t K, const BrickList &B, int64_t limit)
{
    if (limit == 0) return true;
    const volatile BrickSeen *seen = B.seen;
    if (n >= kDenseSorts && seen && seen->n == n && seen->count > 0 && seen->dense >= 0) return 2 * (int64_t)seen->dense > n;
    return n > limit * K;
}
// Granules of a cell from which it alone calls for the digit passes: one workgroup
// puts a cell in order, 18 us for every 1,024 granules.  A cell of 1,024, 2,048, 4,096,
// 16,384 and 65,536 of 262,144 granules, the rest eight a cell, counting: 50, 71, 110,
// 346 and 1,170 us, by digits 68 to 75 (without that cell 36 and 65); of larger beds the
// digit passes cost more.  (At least eight of the samples lie in a cell of n / 512, one
// in any of 2,048 up to eight million granules.)
inline int64_t sort_long(int64_t n) { return 2048 + n / 512; }
// Keys of a tile of a digit pass, in threads: small sorts take small tiles, to
// spread over the chip.
constexpr int kSortThreads = 256, kSortItems = 8;
inline int sort_items(int64_t n) { return n <= kSmallSort ? 1 : kSortItems; }
inline int64_t sort_tiles(int64_t n)
{
    const int64_t keys = (int64_t)kSortThreads * sort_items(n);
    return (n + keys - 1) / keys;
}
inline int64_t sort_tiles_max(int64_t n_max)  // of any n up to n_max
{
    const int64_t a = sort_tiles(n_max), b = sort_tiles(n_max < kSmallSort ? n_max : kSmallSort);
    return a > b ? a : b;
}
inline int sort_passes(int64_t K)
{
    int p = 1;
    while (p < 4 && ((K - 1) >> (8 * p)) != 0) ++p;
    return p;
}

// nl: the neighbour list of the stepping path, or NULL.  With nl, the key
// kernel also measures every granule's displacement since the list's build
// (x in the order of that build) and the sort decides nl->ctl[0]: rebuild
// when force is set, when the sorted order changes, or when a granule moved
// by more than the list's skin / 2.
// B becomes the list of the tables' occupied bricks.
// keep_ranges: cell_begin, cell_end hold the ranges of the last sort on S
// (same n) and B their bricks; they are then rewritten only if a key changed.
hipError_t launch_sort_cells(const DevParams &P, int64_t n, const double *x, uint32_t *key, int32_t *order,
                             int32_t *cell_begin, int32_t *cell_end, int64_t K, SortScratch &S, BrickList &B,
                             int64_t *err, hipStream_t s, const NbrList *nl = nullptr, int force = 1, int keep_ranges = 0);
// Sort of a rollout step (n > 0): xv holds x then v (6 n) in input order; the
// state goes to xvs and rs in sorted order, fx (len int64) is cleared and the
// largest granule fractions of *nb workgroups go to part; with gxv (the reverse
// step) the adjoint of the state goes to gs, moved through the integration, that
// of the force to gF, and gmax is cleared.
hipError_t launch_rollout_sort(const DevParams &P, int64_t n, const double *xv, const double *r, uint32_t *key,
                               int32_t *order, int32_t *cell_begin, int32_t *cell_end, int64_t K, SortScratch &S,
                               BrickList &B, int64_t *err, double *xvs, double *rs, int64_t *fx, int64_t len,
                               double *part, int *nb, const double *gxv, double *gs, double *gF,
                               unsigned long long *gmax, hipStream_t s);
hipError_t launch_rollout_p2g(const DevParams &P, int64_t n, int64_t K, const double *x, const double *r,
                              const int32_t *cb, const int32_t *ce, const BrickList &B, int64_t *fx, double *part, int nb,
                              hipStream_t s);
const double *rollout_scale(const double *part);  // the inverse scale of its sums (device)
hipError_t launch_rollout_galpha(const DevParams &P, int64_t n, int64_t K, const double *x, const double *gaf,
                                 const int32_t *cb, const int32_t *ce, const BrickList &B, const int64_t *fx,
                                 int64_t *fx2, double *part, const unsigned long long *gmax, hipStream_t s);
hipError_t launch_rollout_pull(const DevParams &P, int64_t n, const int32_t *order, const double *x, const double *r,
                               const int64_t *fx2, const unsigned long long *gmax, const double *gs, double *gxv,
                               const double *psum, const BrickList &B, int parts, double *gmu, double *gcd, hipStream_t s);
hipError_t launch_reorder(int64_t n, const int32_t *order, const double *x, const double *v, const double *r,
                          const int32_t *id, double *xo, double *vo, double *ro, int32_t *ido, hipStream_t s);

// The largest brick shell (granule slots, pads included) that the direct
// contact kernel met: dev[2] (device, alternating between recording calls: one
// records into dev[par] and clears dev[par ^ 1]; an atomic maximum, taken only
// when the word is smaller), host (pinned: a copy of the record, read by later
// calls without waiting; 0 until the first copy lands).  Only every 16th call
// records and copies (a copy costs a few microseconds of the stream).  The
// next launches are shaped from the record; a brick beyond the shape takes a
// slower path with the same bits, and the calls after adapt.
struct SizeRecord {
    int32_t *dev;
    int32_t *host;
    int par;
    unsigned calls;
};
// Whether this call copies its record to the host.
inline bool record_copy(SizeRecord *r)
{
    return r && r->host && (r->calls++ & 15u) == 0u;
}

// The granules that an occupied brick holds on average, for the shape of the
// brick kernels: from the last count of occupied bricks that reached the host
// (every 16th list copies it, and the first after one of another number of
// granules; read without waiting), or, before the first of n granules (known
// false), the granules of radius r_max that its 64 cells hold on a cubic lattice.
struct BrickFill {
    double avg;
    bool known;
    double full;  // occupied bricks of a group that holds granules, 0 where not known
    double bricks(int64_t n) const { return (double)n / avg; }
};
inline BrickFill brick_fill(const DevParams &P, int64_t n, const BrickList &B)
{
    const volatile BrickSeen *seen = B.seen;
    const int32_t count = seen && seen->n == n ? seen->count : 0;
    if (count > 0) return {(double)n / count, true, seen->groups > 0 ? (double)seen->bricks / seen->groups : 0.0};
    const double e = 0.5 * P.cell / P.r_max;
    return {kBrickCells * ((e * e) * e), false, 0.0};
}
// How the gather, the direct contact and the direct P2G run.
//
// One wave per brick (workgroups of 64 threads) instead of 256 threads: a
// 256-thread workgroup leaves three of its four waves idle when a brick holds
// about one granule per lane of a wave, and the chip holds a quarter of the
// bricks: 16.8 million granules at 64 a brick take 0.88, 1.04 and 0.92 ms
// instead of 1.25, 1.88 and 1.70 (gather, contact, P2G, FP32); at 205 a brick
// the wave loops over its brick and takes 25 and 32 us instead of 19 and 26
// (gather, P2G).  Beds of fewer granules than fill a wave in each of the 1,024
// larger workgroups that the chip holds (65,536) leave it room, and more threads
// per brick are faster (216 bricks of 64: 7.8 and 7.2 against 6.4 and 6.5 us; 1,728:
// 11.0 and 12.8 against 11.9 and 15.4).
//
// A workgroup of kGroupNT threads per group of 2x2x2 bricks, a wave per brick
// and two bricks per wave, when there are many more bricks: eight tiles share
// their halos (10^3 nodes instead of 8 x 6^3 at a cell of one node spacing), so
// the tiles take 0.58 of the bytes, and so do the cells of eight shells.  The
// same bed, one wave per brick against groups: gather 0.88 and 0.62 ms, contact
// 0.94 and 0.87, P2G 0.90 and 0.68, assembly of the tiles 0.96 and 0.47.  (A
// wave per brick, groups of 512 threads: 0.79, 1.08, 0.91, 0.46: two such
// workgroups fill a CU and wait for each other's loads.)  From 4,096 bricks for
// the node tiles (gather, P2G and assembly there: 15.2 + 17.8 + 10.6 against
// 15.8 + 17.7 + 14.7 us); the contact and the FP64 gather, whose workgroups
// hold more registers and LDS, from 16,384 (8,820 bricks: 42 against 35 us and
// 40 against 34; 13,824: 50 against 51; 18,432: 78.4 against 78.0; 65,536: 231
// against 261 and 226 against 257).  And where a group that holds granules holds
// five of its eight bricks or more: fewer do not share enough.  Steps in FP32 by
// waves against groups: columns of single bricks (two of eight) 285 and 456 us,
// bricks at random, a quarter of the box 292 and 375, 3/8 400 and 492, half 482
// and 535, three quarters 671 and 612; sheets one brick thick (four of eight)
// 398 and 392, 507 and 567, 638 and 606 us, normal to z, x and y.
//
// kFillBoth: not known yet (a first call) and plausible: both kernels are
// launched and the device's count of occupied bricks picks one.
constexpr int64_t kWaveFill = 80;
constexpr int64_t kWaveBricks = 1024;
constexpr int64_t kGroupBricks = 4096;
constexpr int64_t kGroupShells = 16384;
constexpr double kGroupFull = 5.0;
constexpr int kGroupNT = 256;
enum FillMode { kFillBlock = 0, kFillWave = 1, kFillBoth = 2, kFillGroup = 3 };
// least: occupied bricks from which the caller takes groups.
inline FillMode fill_mode(const DevParams &P, int64_t n, const BrickList &B, int64_t least)
{
    const BrickFill f = brick_fill(P, n, B);
    if (f.avg > kWaveFill || n < kWaveBricks * kBrickCells) return kFillBlock;
    if (!f.known) return kFillBoth;
    return (double)n >= (double)least * f.avg && f.full >= kGroupFull ? kFillGroup : kFillWave;
}
template <typename T>
hipError_t launch_contact(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                          const int32_t *cb, const int32_t *ce, const BrickList &B, const T *sr, const double *held,
                          T *F, int32_t *ncont, int64_t *err, hipStream_t s, SizeRecord *ss = nullptr);
// Neighbour-list build (only when force is set or the sort asked for it)
// and the contact forces from the list (Sec. 3.1, Eq. 1a-1c, walls).
// pairs (optional, pair_cap x n, column-major): the partners that touch, in
// the order their forces are summed, -1 after the last.
hipError_t launch_nbr_build(const DevParams &P, int64_t n, const double *x, const double *r, const int32_t *cb,
                            const int32_t *ce, const BrickList &B, NbrList &L, int force, int64_t *err,
                            hipStream_t s);
template <typename T>
hipError_t launch_contact_list(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                               const int32_t *cb, const int32_t *ce, const NbrList &L, T *F, int32_t *ncont,
                               int32_t *pairs, int pair_cap, int64_t *err, hipStream_t s);

template <typename T>
hipError_t launch_g2p(const DevParams &P, int64_t n, const double *x, const T *u, const int64_t *afx,
                      const double *are, T *uat, T *af, hipStream_t s);
template <typename T>
hipError_t launch_moisture_ratio(int64_t n, const double *held, const T *af, T *sr, hipStream_t s);
template <typename T>
hipError_t launch_drag(const DevParams &P, int64_t n, const double *r, const double *v, const T *uat, const T *af,
                       T *Fd, hipStream_t s);
template <typename T>
hipError_t launch_integrate(const DevParams &P, int64_t n, const double *r, const T *Fc, const T *Fd, double *x,
                            double *v, hipStream_t s);

// Scratch of the assembled P2G of the stepping path: one node tile (4
// channels) per occupied brick, and the list of granules whose stencil left
// their brick's tile (at most n) with its counter.
struct P2GStore {
    unsigned long long *tiles;  // [occupied bricks][4][tile nodes]
    int32_t *esc;               // [n]
    uint32_t *esc_n;            // [1] granules listed
    const int32_t *cover;       // per axis and node: (brick, node in its tile) twice, -1 for none
    // per node row (j, k) and segment of 4 nodes along x (row-major, (n0 + 3) / 4
    // segments a row): 1 where the grids may hold a nonzero value, i.e. a
    // tile reached the segment at the last assembly or a listed granule was
    // deposited there since; NULL: every node is written
    uint8_t *live;
    const int32_t *gcover;  // cover of the brick groups' tiles, NULL: no room for those
    int32_t *gslot;         // [groups] the group's tile (its number), -1: no granules
    // set by p2g_store_mode for both launches of a call:
    bool direct;            // the direct kernel, in mode (kFillGroup: the tiles are the groups'), or the run kernel
    FillMode mode;
    int full;  // 1: write every node (the grids hold no earlier assembly's values)
};
// The table P2GStore::cover for the parameters P (host; 4 (n0 + n1 + n2)
// int32): for node i of axis a, at 4 (n0 + ... + n_{a-1} + i), the bricks
// along the axis whose tile holds the node, with the node's offset in it.
// (edge kGroup: of the brick groups and their tiles.)
void p2g_cover_table(const DevParams &P, int edge, int32_t *out);
// Integrate + P2G of the stepping path (dry, alpha and momentum) in two
// launches: launch_integrate_p2g_store moves the granules and stores each
// occupied brick's tile (listing the granules whose stencil left it);
// launch_p2g_assemble then writes the grids from the tiles (written, not
// added to: alpha and mom need no clearing) and deposits the listed
// granules.  esc_next: the escape counter of the next call, cleared here.
// With st.live and !st.full the grids hold the previous assembly's result
// (and its deposits): segments that no tile reaches now and that were not
// live are zero already and are not written again.
void p2g_store_mode(const DevParams &P, int64_t n, const BrickList &B, P2GStore &st);
template <typename T>
hipError_t launch_integrate_p2g_store(const DevParams &P, int64_t n, int64_t K, double *x, double *v,
                                      const double *r, const T *Fc, const T *Fd, const int32_t *cb,
                                      const int32_t *ce, const BrickList &B, int64_t *err, hipStream_t s,
                                      const P2GStore &st);
hipError_t launch_p2g_assemble(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                               const BrickList &B, int64_t *alpha, int64_t *mom, int64_t *err, hipStream_t s,
                               const P2GStore &st, uint32_t *esc_next);

hipError_t launch_fill_i64(int64_t *a, int64_t len, hipStream_t s);
hipError_t launch_fill_f64(double *a, int64_t len, hipStream_t s);
hipError_t launch_p2g_fixed(const DevParams &P, int64_t n, int64_t K, const double *x, const double *v,
                            const double *r, const int32_t *cb, const int32_t *ce, const BrickList &B,
                            int64_t *alpha, int64_t *mom, int64_t *err, hipStream_t s);
template <typename T>
hipError_t launch_integrate_p2g(const DevParams &P, int64_t n, int64_t K, double *x, double *v, const double *r,
                                const T *Fc, const T *Fd, const int32_t *cb, const int32_t *ce, const BrickList &B,
                                int64_t *alpha, int64_t *mom, int64_t *err, hipStream_t s,
                                const double *held = nullptr);  // held: water per granule volume (wet mass), or NULL
// Exchange deposit of one sub-step (Sec. 5.2) into the 3 x G int64 grid fs.
template <typename T>
hipError_t launch_exchange_p2g(const DevParams &P, int64_t n, int64_t K, const double *x, const double *r,
                               const T *Fc, const T *Ffl, const int32_t *cb, const int32_t *ce, const BrickList &B,
                               double exsc, int64_t *fs, int64_t *err, hipStream_t s,
                               const double *held = nullptr);  // held: wet mass and volume, or NULL
template <typename T>
hipError_t launch_gather_g2p_fluid(const DevParams &P, int64_t n, int64_t K, const int32_t *order, const double *x,
                                   const double *v, const double *r, const int32_t *id, double *xo, double *vo,
                                   double *ro, int32_t *ido, const T *u, const int64_t *afx, const T *gp,
                                   const T *fa, const int32_t *cb, const int32_t *ce, const BrickList &B, T *Ff,
                                   hipStream_t s, const double *held = nullptr, double *heldo = nullptr);
template <typename T>
hipError_t launch_gather_g2p_drag(const DevParams &P, int64_t n, int64_t K, const int32_t *order, const double *x,
                                  const double *v, const double *r, const int32_t *id, double *xo, double *vo,
                                  double *ro, int32_t *ido, const T *u, const int64_t *afx, const int32_t *cb,
                                  const int32_t *ce, const BrickList &B, T *Fd, T *uat, T *af, hipStream_t s);
// Unquantised P2G (alpha G, momentum 3G doubles; = or += with acc),
// summed deterministically as integers at a scale set by the largest
// contribution; fx: 4 G int64 and part: 4 x 1024 + 8 doubles of scratch.
hipError_t launch_p2g_real(const DevParams &P, int64_t n, int64_t K, const double *x, const double *v,
                           const double *r, const int32_t *cb, const int32_t *ce, const BrickList &B,
                           double *alpha, double *mom, int acc, int64_t *fx, double *part, hipStream_t s);
hipError_t launch_g2p_vjp_grid(const DevParams &P, int64_t n, int64_t K, const double *x, const double *A,
                               const double *gaf, const int32_t *cb, const int32_t *ce, const BrickList &B,
                               double *gA, int64_t *fx, double *part, hipStream_t s);

// What the differentiable form's kinds of the direct contact kernel (see
// ContactKind in contact.hip) read and write besides the contact's arrays.
struct AdjArgs {
    const double *gF;            // pullbacks: cotangent of the force
    double *gx, *gv, *gmu;       // gic_contact_forces_vjp: added to, added to, written
    const double *u, *inv;       // rollout: fluid velocity; inverse scale of fx
    const int64_t *fx;           // rollout: the alpha deposit's integer sums
    const int32_t *order;        // forward step: sorted position to input index
    double *out;                 // forward step: (x, v) advanced, input order
    double *gs;                  // reverse step: adjoint of (x, v), sorted, in and out
    double *gaf;                 // reverse step: cotangent of the fluid fraction
    unsigned long long *gmax;    // reverse step: bits of the largest |gaf|
    double *psum;                // reverse step: per brick (or workgroup), the sums of dL/dmu and dL/dC_d
    int both;                    // reverse step: both forms were launched, the count of bricks picks one
    int tile_at;                 // rollout: where the brick's node tile lies in LDS (bytes), 0 for none (set at the launch)
};
// Whether the contact pullback runs over the bricks (and reads their list).
bool contact_vjp_bricks(const DevParams &P, int64_t n, const BrickList &B);
hipError_t launch_contact_vjp(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                              const int32_t *cb, const int32_t *ce, const BrickList &B, const AdjArgs &A, int64_t *err,
                              hipStream_t s, SizeRecord *ss, bool bricks);
hipError_t launch_rollout_contact(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                                  const int32_t *cb, const int32_t *ce, const BrickList &B, const AdjArgs &A,
                                  bool reverse, int64_t *err, hipStream_t s, SizeRecord *ss, int *parts = nullptr);
// (*parts: how many sums of the parameter gradients a reverse step leaves in psum:
// one per workgroup of 256 granules, that many; one per occupied brick, 0; the
// number negated where the device picks, see pull_granules)
hipError_t launch_drag_vjp(const DevParams &P, int64_t n, const double *r, const double *v, const double *uat,
                           const double *af, const double *gF, double *gv, double *guat, double *gaf, double *gcd,
                           hipStream_t s);
hipError_t launch_integrate_vjp(const DevParams &P, int64_t n, const double *r, const double *gx, double *gv,
                                double *gF, hipStream_t s);
hipError_t launch_g2p_vjp(const DevParams &P, int64_t n, int64_t K, const double *x, const double *u,
                          const double *A, const double *guat, const double *gaf, const int32_t *cb,
                          const int32_t *ce, const BrickList &B, double *gx, double *gA, int64_t *fx, double *part,
                          hipStream_t s);
hipError_t launch_p2g_vjp(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                          const double *gA, const double *gP, double *gx, double *gv, hipStream_t s);
hipError_t launch_sum(const double *a, const double *b, int64_t n, double *part, int nparts, double *out, int acc,
                      hipStream_t s);
hipError_t launch_permute(int64_t n, int comps, const int32_t *order, const double *in, double *out, int scatter,
                          hipStream_t s);
hipError_t launch_scale(int64_t n, const double *a, const double *sp, double factor, double *out, hipStream_t s);

inline unsigned grid_for(int64_t n, int threads)
{
    int64_t b = (n + threads - 1) / threads;
    return (unsigned)(b < 1 ? 1 : b);
}

}  // namespace gic
