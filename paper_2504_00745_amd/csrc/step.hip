// Fused stages of one sub-step (Alg. 2) on gfx950: the gather into sorted
// order together with G2P (Sec. 5.2) and the drag (Sec. 3.3 Eq. 5b, App. A),
// one workgroup per brick of 4x4x4 cells.  The brick's node tile of fluid
// velocity and clamped solid fraction is copied into LDS once, so each
// granule's 27 node reads come from LDS instead of 4 x 27 global loads.
// Results are bit-identical to the separate reorder, G2P and drag kernels:
// the arithmetic is the same device functions in the same order.
#include "gic_launch.hpp"

namespace gic {

namespace {

// Node tile entry of the drag gather: u and the clamped solid fraction of a
// node, read with one LDS access.
template <typename T>
struct Node4;
template <>
struct Node4<float> {
    using type = float4;
};
template <>
struct Node4<double> {
    using type = double4;
};

// The extra node field e of the fluid gather, a record of its own so that
// the first keeps its one 16-byte (32 in double) access.
template <typename T>
struct Node3 {
    T x, y, z;
};

// g2p_sample_st for a stencil that lies inside the tile: the same weights,
// products and summation order, the node read from the tile at
// lz[cz] + ly[cy] + lx[cx]; EXTRA: e is summed into ea with the same weights.
template <typename T, bool EXTRA, typename V4>
__device__ inline void g2p_sample_tile(const Stencil &s, const V4 *__restrict__ tile,
                                       const Node3<T> *__restrict__ etile, const int lx[3], const int ly[3],
                                       const int lz[3], T uat[3], T &af, T ea[3])
{
    T acc[3] = {(T)0, (T)0, (T)0};
    T as = (T)0;
#pragma unroll
    for (int cz = 0; cz < 3; ++cz) {
        const double wz = s.w[2][cz];
#pragma unroll
        for (int cy = 0; cy < 3; ++cy) {
            const double wyz = s.w[1][cy] * wz;
#pragma unroll
            for (int cx = 0; cx < 3; ++cx) {
                const T w = (T)(s.w[0][cx] * wyz);
                const int k = lz[cz] + ly[cy] + lx[cx];
                const V4 q = tile[k];
                acc[0] += w * q.x;
                acc[1] += w * q.y;
                acc[2] += w * q.z;
                as += w * q.w;
                if (EXTRA) {
                    const Node3<T> e = etile[k];
                    ea[0] += w * e.x;
                    ea[1] += w * e.y;
                    ea[2] += w * e.z;
                }
            }
        }
    }
    uat[0] = acc[0];
    uat[1] = acc[1];
    uat[2] = acc[2];
    af = (T)1 - as;
}

// The gather of one brick per workgroup of NT threads.
//
// FLUID: the remaining interphase forces (Sec. 3.3 Eq. 5a-5c) are added to
// the drag: -V grad p at the granule, plus (rho_f V / 2) a_f under virtual
// mass (the a_s part of the virtual-mass force sits in the effective mass of
// the integrator).  Both are V times the interpolation of one node field,
// e = -grad p + (rho_f / 2) a_f, so the node tile holds e (three channels, a
// second record per node) instead of grad p and a_f (six), sampled in the
// same pass over the 27 nodes with the same weights as u and alpha.  For wet
// granules (held given, in the input order) V = (4/3) pi r^3 (1 + held): the
// absorbed water counts as volume (Sec. 5.3); held is gathered into heldo
// with the rest of the state.
// The second record is read in place of seven scalar reads per node, and the
// first granule's state is fetched before the tile: a 1.05 million granule
// column 73 -> 50 us (FP32), 0.52 million wet granules 48 -> 29 us.
template <typename T, bool FLUID, int NT, bool GROUP>
__global__ void __launch_bounds__(NT) k_gather(DevParams P, int64_t n, const int32_t *__restrict__ bl,
                                               const int32_t *__restrict__ bcnt, const int32_t *__restrict__ order,
                                               const double *__restrict__ x, const double *__restrict__ v,
                                               const double *__restrict__ r, const int32_t *__restrict__ id,
                                               double *__restrict__ xo, double *__restrict__ vo,
                                               double *__restrict__ ro, int32_t *__restrict__ ido,
                                               const T *__restrict__ u, const int64_t *__restrict__ afx,
                                               const T *__restrict__ gp, const T *__restrict__ fa,
                                               const int32_t *__restrict__ cb, const int32_t *__restrict__ ce,
                                               T *__restrict__ Ff, T *__restrict__ uat, T *__restrict__ af,
                                               const double *__restrict__ held, double *__restrict__ heldo, int only)
{
    using V4 = typename Node4<T>::type;
    extern __shared__ double smem_d[];
    if (not_mine(only, kWaveFill, n, bcnt)) return;
    constexpr int kBricks = GROUP ? kGroup * kGroup * kGroup : 1;
    __shared__ int32_t s_beg[kBricks], s_end[kBricks];  // GROUP: its bricks' granules
    const int tid = threadIdx.x;
    int64_t b;             // the tile's (first) brick
    int32_t gb = 0, ge = 0;
    if (GROUP) {
        const Group grp = group_of_block(P);
        if (grp.id < 0) return;
        b = brick_of_group(P, grp, 0);
        const int64_t t = tid < kBricks ? brick_of_group(P, grp, tid) : -1;
        if (t >= 0) {
            gb = cb[t * kBrickCells];
            ge = ce[t * kBrickCells + kBrickCells - 1];
            clip_range(n, gb, ge);
        }
        if (tid < kBricks) {
            s_beg[tid] = gb;
            s_end[tid] = ge;
        }
        if (!__syncthreads_or(gb < ge)) return;
        gb = s_beg[tid >> 6];
        ge = s_end[tid >> 6];
    } else {
        b = brick_of_block(bl, bcnt);
        if (b < 0) return;
        gb = cb[b * kBrickCells];
        ge = ce[b * kBrickCells + kBrickCells - 1];
        clip_range(n, gb, ge);
        if (ge <= gb) return;
    }
    constexpr int kStep = GROUP ? 64 : NT;  // threads on a brick
    const int64_t q0 = (int64_t)gb + tid % kStep;  // the thread's first granule
    const int E = GROUP ? P.gtile : P.tile, E3 = E * E * E;
    const int64_t G = P.G;
    V4 *su = reinterpret_cast<V4 *>(smem_d);                   // [E3]: u_x, u_y, u_z, clamped alpha
    Node3<T> *se = reinterpret_cast<Node3<T> *>(su + E3);      // [E3]: e (FLUID)
    const bool vm_acc = FLUID && P.vmass && fa != nullptr;
    const bool extra = FLUID && (gp || vm_acc);
    const T half_rho_f = (T)P.half_rho_f;
    // e = -grad p + (rho_f / 2) a_f at grid node idx, component c
    auto extra_field = [&](int c, int64_t idx) {
        T e = gp ? -gp[c * G + idx] : (T)0;
        if (vm_acc) e = e + half_rho_f * fa[c * G + idx];
        return e;
    };
    int32_t o[3];
    tile_origin(P, b, o);
    // the first granule's state is fetched before the tile, so the two
    // loads' latencies overlap
    int64_t s = -1;
    double xa[3] = {0.0, 0.0, 0.0}, va[3] = {0.0, 0.0, 0.0}, rq = 0.0, hq = 0.0;
    int32_t idq = 0;
    auto fetch = [&](int64_t q) {
        s = order[q];
        if ((uint64_t)s >= (uint64_t)n) return;
        for (int a = 0; a < 3; ++a) {
            xa[a] = x[a * n + s];
            va[a] = v[a * n + s];
        }
        rq = r[s];
        if (ido) idq = id[s];
        if (FLUID && held) hq = held[s];
    };
    if (q0 < ge) fetch(q0);
    for (int k = threadIdx.x; k < E3; k += NT) {
        const int32_t i = o[0] + k % E, j = o[1] + (k / E) % E, l = o[2] + k / (E * E);
        if (i < 0 || j < 0 || l < 0 || i >= P.n[0] || j >= P.n[1] || l >= P.n[2]) continue;  // never referenced
        const int64_t idx = node_index(P, i, j, l);
        V4 q;
        q.x = u[idx];
        q.y = u[G + idx];
        q.z = u[2 * G + idx];
        q.w = (T)node_alpha(P, afx[idx]);
        su[k] = q;
        if (extra) {
            Node3<T> e;
            e.x = extra_field(0, idx);
            e.y = extra_field(1, idx);
            e.z = extra_field(2, idx);
            se[k] = e;
        }
    }
    __syncthreads();
    // fetched: granule q's state is the one fetched before the tile.  Its place does
    // not tell: an empty first brick begins where the wave's next brick does.
    auto gather = [&](int64_t q, bool fetched) {
        if (!fetched) fetch(q);
        if ((uint64_t)s >= (uint64_t)n) return;  // not a permutation of [0, n): position q left untouched
        for (int a = 0; a < 3; ++a) {
            xo[a * n + q] = xa[a];
            vo[a * n + q] = va[a];
        }
        ro[q] = rq;
        if (ido) ido[q] = idq;
        if (FLUID && heldo) heldo[q] = hq;
        Stencil st;
        stencil_of(P, xa, st);
        // tile offsets of the stencil's nodes; every node inside the tile is
        // the rule (a granule outside its brick's tile only if its cell is
        // clamped)
        int lx[3], ly[3], lz[3];
        bool inside = true;
        for (int k = 0; k < 3; ++k) {
            const int ax = st.node[0][k] - o[0], ay = st.node[1][k] - o[1], az = st.node[2][k] - o[2];
            inside &= ax >= 0 && ay >= 0 && az >= 0 && ax < E && ay < E && az < E;
            lx[k] = ax;
            ly[k] = ay * E;
            lz[k] = az * E * E;
        }
        T ua[3], a;
        T ea[3] = {(T)0, (T)0, (T)0};
        if (inside) {
            if (extra)
                g2p_sample_tile<T, true>(st, su, se, lx, ly, lz, ua, a, ea);
            else
                g2p_sample_tile<T, false>(st, su, se, lx, ly, lz, ua, a, ea);
        } else {
            int t = -1;        // tile slot of the node just fetched, -1 outside the tile
            int64_t gidx = 0;  // its grid index when outside
            g2p_sample_st<T>(st, [&](int32_t i, int32_t j, int32_t k, T uu[3], T &al) {
                const int32_t li = i - o[0], lj = j - o[1], lk = k - o[2];
                t = -1;
                if (li >= 0 && lj >= 0 && lk >= 0 && li < E && lj < E && lk < E) {
                    t = (lk * E + lj) * E + li;
                    const V4 w = su[t];
                    uu[0] = w.x;
                    uu[1] = w.y;
                    uu[2] = w.z;
                    al = w.w;
                } else {
                    gidx = node_index(P, i, j, k);
                    uu[0] = u[gidx];
                    uu[1] = u[G + gidx];
                    uu[2] = u[2 * G + gidx];
                    al = (T)node_alpha(P, afx[gidx]);
                }
            }, ua, a, [&](T w) {
                if (!extra) return;
                const Node3<T> e = t >= 0 ? se[t] : Node3<T>{extra_field(0, gidx), extra_field(1, gidx),
                                                             extra_field(2, gidx)};
                ea[0] += w * e.x;
                ea[1] += w * e.y;
                ea[2] += w * e.z;
            });
        }
        T f[3];
        drag_one<T>(P, rq, va, ua, a, f);
        if (extra) {
            const T tV = (T)wet_volume(rq, hq);
            for (int c = 0; c < 3; ++c) f[c] = f[c] + tV * ea[c];
        }
        for (int c = 0; c < 3; ++c) Ff[c * n + q] = f[c];
        if (uat) {
            uat[q] = ua[0];
            uat[n + q] = ua[1];
            uat[2 * n + q] = ua[2];
        }
        if (af) af[q] = a;
    };
    for (int64_t q = q0; q < ge; q += kStep) gather(q, q == q0);
    if (GROUP)
        for (int w = (tid >> 6) + NT / 64; w < kBricks; w += NT / 64)
            for (int64_t q = (int64_t)s_beg[w] + (tid & 63); q < s_end[w]; q += 64) gather(q, false);
}

// Threads per workgroup: see fill_mode.
template <typename T, bool FLUID>
hipError_t launch_gather(const DevParams &P, int64_t n, int64_t K, const int32_t *order, const double *x,
                         const double *v, const double *r, const int32_t *id, double *xo, double *vo, double *ro,
                         int32_t *ido, const T *u, const int64_t *afx, const T *gp, const T *fa, const int32_t *cb,
                         const int32_t *ce, const BrickList &B, T *Ff, T *uat, T *af, const double *held,
                         double *heldo, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const unsigned grid = brick_grid(K / kBrickCells);
    const size_t node = sizeof(T) * (FLUID ? 7 : 4);
    const size_t lds = node * P.tile * P.tile * P.tile, glds = node * P.gtile * P.gtile * P.gtile;
    constexpr int kGatherNT = sizeof(T) == 4 ? kGroupNT : 128;
    FillMode mode = fill_mode(P, n, B, sizeof(T) == 4 ? kGroupBricks : kGroupShells);
    // the FP64 fluid tile of a group leaves a CU two workgroups
    if (mode == kFillGroup && ((FLUID && sizeof(T) == 8) || glds > 65536)) mode = kFillWave;
#define GIC_GATHER(NT, GROUP, ONLY)                                                                           \
    k_gather<T, FLUID, NT, GROUP><<<GROUP ? group_grid(P) : grid, NT, GROUP ? glds : lds, s>>>(               \
        P, n, B.use, B.use_count, order, x, v, r, id, xo, vo, ro, ido, u, afx, gp, fa, cb, ce, Ff, uat, af,   \
        held, heldo, ONLY)
    if (mode == kFillGroup) GIC_GATHER(kGatherNT, true, 0);
    if (mode == kFillWave || mode == kFillBoth) GIC_GATHER(64, false, mode == kFillBoth ? 1 : 0);
    if (mode == kFillBlock || mode == kFillBoth) GIC_GATHER(256, false, mode == kFillBoth ? 2 : 0);
#undef GIC_GATHER
    return hipGetLastError();
}

}  // namespace

template <typename T>
hipError_t launch_gather_g2p_fluid(const DevParams &P, int64_t n, int64_t K, const int32_t *order, const double *x,
                                   const double *v, const double *r, const int32_t *id, double *xo, double *vo,
                                   double *ro, int32_t *ido, const T *u, const int64_t *afx, const T *gp,
                                   const T *fa, const int32_t *cb, const int32_t *ce, const BrickList &B, T *Ff,
                                   hipStream_t s, const double *held, double *heldo)
{
    return launch_gather<T, true>(P, n, K, order, x, v, r, id, xo, vo, ro, ido, u, afx, gp, fa, cb, ce, B, Ff, nullptr,
                                  nullptr, held, heldo, s);
}

template hipError_t launch_gather_g2p_fluid<float>(const DevParams &, int64_t, int64_t, const int32_t *,
                                                   const double *, const double *, const double *, const int32_t *,
                                                   double *, double *, double *, int32_t *, const float *,
                                                   const int64_t *, const float *, const float *, const int32_t *,
                                                   const int32_t *, const BrickList &, float *, hipStream_t,
                                                   const double *, double *);
template hipError_t launch_gather_g2p_fluid<double>(const DevParams &, int64_t, int64_t, const int32_t *,
                                                    const double *, const double *, const double *, const int32_t *,
                                                    double *, double *, double *, int32_t *, const double *,
                                                    const int64_t *, const double *, const double *, const int32_t *,
                                                    const int32_t *, const BrickList &, double *, hipStream_t,
                                                    const double *, double *);

template <typename T>
hipError_t launch_gather_g2p_drag(const DevParams &P, int64_t n, int64_t K, const int32_t *order, const double *x,
                                  const double *v, const double *r, const int32_t *id, double *xo, double *vo,
                                  double *ro, int32_t *ido, const T *u, const int64_t *afx, const int32_t *cb,
                                  const int32_t *ce, const BrickList &B, T *Fd, T *uat, T *af, hipStream_t s)
{
    return launch_gather<T, false>(P, n, K, order, x, v, r, id, xo, vo, ro, ido, u, afx, nullptr, nullptr, cb, ce, B,
                                   Fd, uat, af, nullptr, nullptr, s);
}

template hipError_t launch_gather_g2p_drag<float>(const DevParams &, int64_t, int64_t, const int32_t *,
                                                  const double *, const double *, const double *, const int32_t *,
                                                  double *, double *, double *, int32_t *, const float *,
                                                  const int64_t *, const int32_t *, const int32_t *,
                                                  const BrickList &, float *, float *, float *, hipStream_t);
template hipError_t launch_gather_g2p_drag<double>(const DevParams &, int64_t, int64_t, const int32_t *,
                                                   const double *, const double *, const double *, const int32_t *,
                                                   double *, double *, double *, int32_t *, const double *,
                                                   const int64_t *, const int32_t *, const int32_t *,
                                                   const BrickList &, double *, double *, double *, hipStream_t);

}  // namespace gic
