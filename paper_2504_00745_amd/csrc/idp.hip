// f4: density projection of the fluid fraction (Sec. 5.1, Eq. 12b and 13;
// App. B discretisation on the MAC grid) on gfx950.
//
// Cells are the transfer grid's nodes (cell centres, x fastest).  With the
// scaled pressure q = (dt^2 / (rho_0 dx^2)) p_2, every fluid cell satisfies
//     (L q)_c = sum_j beta_cj (q_c - q_j) = alpha'_c (clamp(alpha*_c / alpha'_c, 0.5, 1.5) - 1),
// beta_cj = (alpha'_c + alpha'_j) / 2 over the six face neighbours that are
// not solid (an air neighbour is a Dirichlet neighbour with q_j = 0; a solid
// neighbour or the box boundary closes the face).  Non-fluid cells are
// identity rows with a zero right-hand side, so L is symmetric positive
// definite on the whole grid and the solution is zero off the fluid.
//
// The solve is conjugate gradients preconditioned by one multigrid V-cycle
// per iteration (the default; Jacobi as the alternative).  The iteration's
// kernels are streaming or blocked stencil passes over the cells (HBM
// bound), the coarse levels launch-latency bound.  Dot products are reduced
// without atomics: each block writes one partial per quantity, and every
// block of the consuming kernel sums all partials in the same fixed order,
// so the iteration is deterministic and needs no clearing between launches.
#include <string.h>

#include "idp_launch.hpp"

namespace gic {

namespace {

constexpr int kIdpThreads = 512;
constexpr int kIdpWaves = kIdpThreads / 64;

__device__ inline double block_sum(double v, double *red)
{
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) red[w] = v;
    __syncthreads();
    double t = red[0];
#pragma unroll
    for (int i = 1; i < kIdpWaves; ++i) t += red[i];
    return t;
}

// Sum of the nb partials of a quantity, identical in every block.
__device__ inline double sum_partials(const double *__restrict__ part, int nb, double *red)
{
    double v = 0.0;
    for (int i = threadIdx.x; i < nb; i += kIdpThreads) v += part[i];
    return block_sum(v, red);
}

// Two such sums at once.
__device__ inline void sum_partials2(const double *__restrict__ p, const double *__restrict__ q, int nb, double *red,
                                     double &s, double &t)
{
    double v = 0.0, u = 0.0;
    for (int i = threadIdx.x; i < nb; i += kIdpThreads) {
        v += p[i];
        u += q[i];
    }
    for (int m = 32; m >= 1; m >>= 1) {
        v += __shfl_xor(v, m);
        u += __shfl_xor(u, m);
    }
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    __syncthreads();
    if (l == 0) {
        red[w] = v;
        red[kIdpWaves + w] = u;
    }
    __syncthreads();
    s = red[0];
    t = red[kIdpWaves];
#pragma unroll
    for (int i = 1; i < kIdpWaves; ++i) {
        s += red[i];
        t += red[kIdpWaves + i];
    }
}

struct Nbr {
    int64_t off;   // index offset of the neighbour
    bool inside;   // within the box
};

// Coordinates of cell c.  Below 2^31 cells the two divisions are a multiply
// by a reciprocal and a shift (the stencil kernels would otherwise spend
// most of their instructions on them); larger grids divide in 64 bits.
__device__ inline void coords(const IdpDims &D, int64_t c, int64_t &i, int64_t &j, int64_t &k)
{
    if (D.G <= 0x80000000ll) {
        const uint32_t cc = (uint32_t)c, nx = (uint32_t)D.nx, ny = (uint32_t)D.ny;
        const uint32_t row = (uint32_t)(((uint64_t)cc * D.mx) >> D.shx);
        i = cc - row * nx;
        const uint32_t kk = (uint32_t)(((uint64_t)row * D.my) >> D.shy);
        j = row - kk * ny;
        k = kk;
    } else {
        const int64_t row = c / D.nx;
        i = c - row * D.nx;
        k = row / D.ny;
        j = row - k * D.ny;
    }
}

// The six face neighbours of cell c = (i, j, k) in the fixed order -x, +x, -y, +y, -z, +z.
__device__ inline void neighbours(const IdpDims &D, int64_t i, int64_t j, int64_t k, Nbr nb[6])
{
    nb[0] = {-1, i > 0};
    nb[1] = {1, i < D.nx - 1};
    nb[2] = {-D.nx, j > 0};
    nb[3] = {D.nx, j < D.ny - 1};
    nb[4] = {-D.sxy, k > 0};
    nb[5] = {D.sxy, k < D.nz - 1};
}

__device__ inline void neighbours(const IdpDims &D, int64_t c, Nbr nb[6])
{
    int64_t i, j, k;
    coords(D, c, i, j, k);
    neighbours(D, i, j, k, nb);
}

// (L v)_c and the diagonal of L at c.
__device__ inline void apply_row(const IdpDims &D, int64_t c, const double *__restrict__ at,
                                 const uint8_t *__restrict__ lab, const double *__restrict__ v, double &Lv,
                                 double &diag)
{
#pragma clang fp contract(off)
    if (lab[c] != kIdpFluid) {
        Lv = v[c];
        diag = 1.0;
        return;
    }
    Nbr nb[6];
    neighbours(D, c, nb);
    const double ac = at[c], vc = v[c];
    double acc = 0.0, dg = 0.0;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        if (!nb[f].inside) continue;
        const int64_t n = c + nb[f].off;
        const uint8_t ln = lab[n];
        if (ln == kIdpSolid) continue;
        const double beta = (ac + at[n]) * 0.5;
        const double vn = ln == kIdpFluid ? v[n] : 0.0;
        acc += beta * (vc - vn);
        dg += beta;
    }
    Lv = acc;
    diag = dg;
}

// sum over the open faces of cell c = (i, j, k) of beta (v_c - v_n), from
// the signed coefficients ac (alpha_f' on fluid cells, -alpha_f' on air
// cells, 0 on solid cells): the six neighbours' coefficients and values are
// loaded without branches; a closed face gets beta = 0 and an air neighbour
// the value 0, so the sum is the operator's for any values v.  val(n, i, j, k)
// gives the value of cell n at (i, j, k).
template <typename V>
__device__ inline double face_sum_ac(const IdpDims &D, int64_t c, int64_t i, int64_t j, int64_t k,
                                     const double *__restrict__ ac, V val)
{
    const int64_t off[6] = {-1, 1, -D.nx, D.nx, -D.sxy, D.sxy};
    const bool in[6] = {i > 0, i < D.nx - 1, j > 0, j < D.ny - 1, k > 0, k < D.nz - 1};
    const int64_t di[6] = {-1, 1, 0, 0, 0, 0}, dj[6] = {0, 0, -1, 1, 0, 0}, dk[6] = {0, 0, 0, 0, -1, 1};
    const double a = ac[c], vc = val(c, i, j, k);
    double an[6], vn[6];
    // a neighbour outside the box reads the cell itself (so that every load is
    // issued without a branch, all before any is used) and gets an = 0: it
    // contributes nothing, whatever vn holds
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const int64_t n = c + (in[f] ? off[f] : 0);
        an[f] = ac[n];
        vn[f] = val(n, in[f] ? i + di[f] : i, in[f] ? j + dj[f] : j, in[f] ? k + dk[f] : k);
    }
#pragma unroll
    for (int f = 0; f < 6; ++f) an[f] = in[f] ? an[f] : 0.0;
    double acc = 0.0;
#pragma unroll
    for (int f = 0; f < 6; ++f) {
        const double beta = an[f] != 0.0 ? (a + fabs(an[f])) * 0.5 : 0.0;
        const double v = an[f] > 0.0 ? vn[f] : 0.0;
        acc += beta * (vc - v);
    }
    return acc;
}

__global__ void __launch_bounds__(kIdpThreads) k_idp_setup(IdpDims D, double alpha_max,
                                                           const int64_t *__restrict__ afx,
                                                           const double *__restrict__ astar,
                                                           const uint8_t *__restrict__ lab, double *__restrict__ at,
                                                           double *__restrict__ s, int64_t *err)
{
#pragma clang fp contract(off)
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        if (lab[c] > kIdpSolid) raise_error(err, kErrRange, c);
        double as = (double)afx[c] * 2.3283064365386963e-10;  // 2^-32
        as = as < alpha_max ? as : alpha_max;
        const double a = 1.0 - as;
        at[c] = a;
        double ratio = astar[c] / a;
        ratio = ratio < 0.5 ? 0.5 : (ratio > 1.5 ? 1.5 : ratio);
        s[c] = lab[c] == kIdpFluid ? a * (ratio - 1.0) : 0.0;
    }
}

__global__ void __launch_bounds__(kIdpThreads) k_idp_apply(IdpDims D, const double *__restrict__ at,
                                                           const uint8_t *__restrict__ lab,
                                                           const double *__restrict__ v, double *__restrict__ out)
{
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        double Lv, dg;
        apply_row(D, c, at, lab, v, Lv, dg);
        out[c] = Lv;
    }
}

// CG start: r = s - L q, z = r / diag (in the partials only), the signed coefficients ac
// (alpha_f' on fluid cells, -alpha_f' on air cells, 0 on solid cells) that
// the iteration kernels read instead of alpha_f' and the labels; partials of
// s.s, r.z, r.r.
__global__ void __launch_bounds__(kIdpThreads) k_cg_init(IdpDims D, const double *__restrict__ at,
                                                         const uint8_t *__restrict__ lab,
                                                         const double *__restrict__ s, const double *__restrict__ q,
                                                         double *__restrict__ r, double *__restrict__ dinv,
                                                         double *__restrict__ ac,
                                                         double *__restrict__ part, CgState *__restrict__ st,
                                                         int64_t *err)
{
    __shared__ double red[kIdpWaves];
    double rz = 0.0, rr = 0.0, ss = 0.0;
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        double Lq, dg;
        apply_row(D, c, at, lab, q, Lq, dg);
        const uint8_t lc = lab[c];
        // the signed coefficients need alpha_f' > 0 on fluid and air cells and a known label
        if (lc > kIdpSolid || (lc != kIdpSolid && !(at[c] > 0.0 && at[c] < INFINITY)))
            raise_error(err, kErrRange, c);
        ac[c] = lc == kIdpFluid ? at[c] : (lc == kIdpAir ? -at[c] : 0.0);
        const double sc = lab[c] == kIdpFluid ? s[c] : 0.0;
        const double rc = sc - Lq;
        const double di = dg > 0.0 ? 1.0 / dg : 0.0;  // a fluid cell walled in on all sides: singular row
        const double zc = rc * di;
        r[c] = rc;
        dinv[c] = di;
        rz += rc * zc;
        rr += rc * rc;
        ss += sc * sc;
    }
    const int nb = gridDim.x;
    rz = block_sum(rz, red);
    rr = block_sum(rr, red);
    ss = block_sum(ss, red);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = ss;
        part[nb + blockIdx.x] = rz;
        part[2 * nb + blockIdx.x] = rr;
        if (blockIdx.x == 0) st->done = -1;  // kernels of a previous solve may have left it set
    }
}

// Reduces the start partials into the scalar state (one block).
__global__ void __launch_bounds__(kIdpThreads) k_cg_start(int nb, const double *__restrict__ part, double tol,
                                                          CgState *__restrict__ st)
{
    __shared__ double red[kIdpWaves];
    const double ss = sum_partials(part, nb, red);
    const double rz = sum_partials(part + nb, nb, red);
    const double rr = sum_partials(part + 2 * nb, nb, red);
    if (threadIdx.x == 0) {
        st->rz[0] = rz;
        st->rz[1] = rz;
        st->ss = ss;
        st->thr = tol * tol * ss;
        st->rr = rr;
        st->done = rr <= tol * tol * ss ? 0 : -1;
        st->iters = 0;
    }
}

// Stencil passes of a conjugate-gradient iteration, blocked in 2.5D; the
// streaming passes around them are fused in, so that each vector is read and
// written as seldom as the iteration allows.
//   kApplyMg, kApplyJac, iteration k: the direction d = z + beta d_old (z from
//     the V-cycle, or r / diag; beta = rz_k / rz_{k-1}, d = z at k = 0), formed
//     as each value is loaded and stored in the other direction buffer (the
//     halo reads d_old), and w = L d; partials of d.w.  Before that the
//     stopping test on the last iteration's r.r.
//   kUpdate, iteration k, multigrid: q += alpha d, r' = r - alpha w (stored in
//     the buffer of z, which d has consumed; partials of r'.r'), the residual
//     r' - A w D^-1 r' of the pre-sweep from zero and its restriction: the
//     coarse right-hand side is the sum of the fluid children's residuals.
//   kResidual: the last part of that, of a level's right-hand side b.
//   kPost: u = w D^-1 b + P E (coarse correction, zero off the coarse fluid)
//     and one sweep, e = u + w D^-1 (b - A u) on fluid cells, b elsewhere; on
//     the finest level the partials of b.e (= r.z).
// A block takes x-y tiles of kTileX x kTileY cells (each wave two adjacent
// rows of 32, so that four lanes hold the four children of a coarse cell in a
// plane) and a run of zlen planes (even).  It keeps its columns' coefficients
// and values for planes z - 1, z, z + 1 in registers and the tile of plane z
// with a one-cell halo in LDS, so that each operand is read from memory about
// once instead of once per neighbour; the next plane of each column and the
// next halo are loaded one step ahead, within the run.  (Tiles of 64 x 8 with
// two rows per thread took 171 registers in kUpdate, two waves per SIMD, and
// a larger halo.)  The face sum is face_sum_ac's, term by term in the same order
// (but for z before y where those are exchanged; cells outside the box hold
// coefficient 0 and value 0).  Items (tile, run of
// planes) are dealt to the blocks; the block count is the other iteration
// kernels', whose partial sums these kernels' must match.
// Bound by HBM: on 4.2 M cells the apply pass takes 32 us (197 MB), the update
// 51 (310 MB with the halo), the post pass 29 (about 160 MB), 6 TB/s each;
// separate direction and product passes took 38, update, residual and
// restriction 69, prolongation and sweep 54, and five more launches.
constexpr double kOmega = 2.0 / 3.0;  // damping of the multigrid's Jacobi sweeps
constexpr int kTileX = 32, kTileY = kIdpThreads / kTileX;
enum StencilMode { kApplyMg, kApplyJac, kUpdate, kResidual, kPost };

// (x, y, z of the pass: the grid's, or with y and z exchanged, see stencil_items)
struct StencilArgs {
    int64_t nx, ny, nz, ry, rz;  // cells per axis; distance of rows and of planes
    int64_t cry, crz;            // of the coarse rows and planes
    int exchanged;
    int ntx, nty, zlen, k;
    double scale;
    const double *ac, *dinv;
    const double *p;       // kApplyMg: z; kApplyJac, kUpdate: r; else: b
    const double *d;       // kApply: the old direction; kUpdate: the direction
    const double *w;       // kUpdate: L d
    const double *ec;      // kPost: the coarse correction
    const double *acc;     // kUpdate, kResidual: the coarse coefficients
    double *o1, *o2;       // outputs: d, w | q, r' | - , - | e
    double *bc;            // kUpdate, kResidual: the coarse right-hand side
    double *part;
    CgState *st;
};

// Off: byte offsets inside a plane, 32 bits where it reaches below 4 GiB (the
// loads then take a scalar base and a 32-bit offset).
template <int MODE, typename Off>
__global__ void __launch_bounds__(kIdpThreads) __attribute__((amdgpu_waves_per_eu(4))) k_stencil(StencilArgs A)
{
    constexpr bool kApply = MODE == kApplyMg || MODE == kApplyJac;
    constexpr bool kRestrict = MODE == kUpdate || MODE == kResidual;
    __shared__ double red[2 * kIdpWaves];
    __shared__ double sa[kTileY + 2][kTileX + 2], sv[kTileY + 2][kTileX + 2];
    __shared__ int64_t s_done;
    // block 0 of an apply pass may set done while others start: read it once per block
    if (threadIdx.x == 0) s_done = A.st->done;
    __syncthreads();
    if (s_done >= 0) return;
    const int64_t nb = gridDim.x;
    const bool first = kApply && A.k == 0;
    double coef = 0.0;  // beta of the apply passes, alpha of the update
    const int tx = threadIdx.x & (kTileX - 1), ty = threadIdx.x / kTileX, t = threadIdx.x;
    const int64_t nx = A.nx, ny = A.ny, nz = A.nz;
    const int64_t tiles = (int64_t)A.ntx * A.nty, nzc = (nz + A.zlen - 1) / A.zlen, items = tiles * nzc;
    // what a cell's coefficient a, value v, right-hand side b and 1 / diag come from
    struct Raw {
        double a, p, s, q;
    };
    auto at = [](const double *base, Off off) {
        return *reinterpret_cast<const double *>(reinterpret_cast<const char *>(base) + off);
    };
    auto put = [](double *base, Off off, double v) {
        *reinterpret_cast<double *>(reinterpret_cast<char *>(base) + off) = v;
    };
    // the cell at off in plane z; its coarse cell at coff in plane z / 2
    auto load = [&](int64_t z, Off off, Off coff) {
        const int64_t pz = z * A.rz;
        Raw r;
        r.a = at(A.ac + pz, off);
        r.p = at(A.p + pz, off);
        r.s = MODE != kApplyMg ? at(A.dinv + pz, off) : 0.0;
        r.q = 0.0;
        if (kApply && !first) r.q = at(A.d + pz, off);
        if (MODE == kUpdate) r.q = at(A.w + pz, off);
        if (MODE == kPost) r.q = at(A.ec + (z >> 1) * A.crz, coff);
        return r;
    };
    const Raw none = {0.0, 0.0, 0.0, 0.0};
    // (coef is set below, after the first loads are under way)
    auto rhs = [&](const Raw &r) { return MODE == kUpdate ? r.p - coef * r.q : r.p; };
    auto value = [&](const Raw &r) {
        if (MODE == kApplyMg) return first ? r.p : r.p + coef * r.q;
        if (MODE == kApplyJac) return first ? r.p * r.s : r.p * r.s + coef * r.q;
        const double e1 = kOmega * r.s * rhs(r);
        return MODE == kPost ? e1 + r.q : e1;
    };
    // halo slot of this thread: rows below and above the tile (t < 64), columns left and right (t < 96)
    int hr = -1, hc = -1, hdi = 0, hdj = 0;
    if (t < kTileX) { hr = 0; hc = t + 1; hdi = t; hdj = -1; }
    else if (t < 2 * kTileX) { hr = kTileY + 1; hc = t - kTileX + 1; hdi = t - kTileX; hdj = kTileY; }
    else if (t < 2 * kTileX + kTileY) { hr = t - 2 * kTileX + 1; hc = 0; hdi = -1; hdj = t - 2 * kTileX; }
    else if (t < 2 * kTileX + 2 * kTileY) { hr = t - 2 * kTileX - kTileY + 1; hc = kTileX + 1; hdi = kTileX; hdj = t - 2 * kTileX - kTileY; }
    // items in tile order within a run of planes; workgroups are dealt to the
    // eight XCDs in turn, so block b starts at item (b % 8) nb/8 + b/8 and each
    // XCD takes a contiguous eighth (y-adjacent tiles share its L2)
    const int64_t it0 = nb % 8 ? (int64_t)blockIdx.x : (blockIdx.x % 8) * (nb / 8) + blockIdx.x / 8;
    double dot = 0.0;
    int64_t z0 = 0, z1 = 0, i = 0, j = 0;
    bool own = false, hown = false;
    Off col = 0, ccol = 0, hcol = 0, hccol = 0;
    Raw rm = none, r0 = none, rp = none, h = none;
    auto plane = [&](int64_t z) { return own && z >= 0 && z < nz ? load(z, col, ccol) : none; };
    auto begin = [&](int64_t it) {  // an item's place and its first loads
        const int64_t tile = it % tiles;
        z0 = (it / tiles) * A.zlen;
        z1 = z0 + A.zlen < nz ? z0 + A.zlen : nz;
        const int64_t i0 = (tile % A.ntx) * kTileX, j0 = (tile / A.ntx) * kTileY;
        i = i0 + tx;
        j = j0 + ty;
        own = i < nx && j < ny;
        col = own ? (Off)(j * A.ry + i) * 8 : 0;
        ccol = own ? (Off)((j >> 1) * A.cry + (i >> 1)) * 8 : 0;
        const int64_t hi = i0 + hdi, hj = j0 + hdj;
        hown = hr >= 0 && hi >= 0 && hi < nx && hj >= 0 && hj < ny;
        hcol = hown ? (Off)(hj * A.ry + hi) * 8 : 0;
        hccol = hown ? (Off)((hj >> 1) * A.cry + (hi >> 1)) * 8 : 0;
        rm = plane(z0 - 1);
        r0 = plane(z0);
        rp = plane(z0 + 1);
        h = hown ? load(z0, hcol, hccol) : none;
    };
    // (kUpdate begins after alpha is known: held over the sum, its first loads
    // cost registers beyond 128 and 7 us of 51)
    if (MODE != kUpdate && it0 < items) begin(it0);
    if (kApply && !first) {
        const double thr = A.st->thr, rz0 = A.st->rz[(A.k + 1) & 1];
        double rz1, rr;
        sum_partials2(A.part + nb, A.part + 2 * nb, (int)nb, red, rz1, rr);
        const bool conv = rr <= thr;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            A.st->rz[A.k & 1] = rz1;
            A.st->rr = rr;
            A.st->iters = A.k;
            if (conv) A.st->done = A.k;
        }
        if (conv) return;
        coef = rz1 / rz0;
    }
    if (MODE == kUpdate) {
        const double rz = A.st->rz[A.k & 1];
        coef = rz / sum_partials(A.part, (int)nb, red);
    }
    for (int64_t it = it0; it < items; it += nb) {
        if (MODE == kUpdate || it != it0) begin(it);
        // the column: m = z - 1, 0 = z, p = z + 1; halo of plane z
        double am = rm.a, vm = value(rm), a0 = r0.a, v0 = value(r0), ap = rp.a, vp = value(rp);
        double b0 = rhs(r0), bp = rhs(rp), s0 = r0.s, sp = rp.s;  // right-hand side, 1 / diag
        double half = 0.0;                                        // kRestrict: the even plane's children
        for (int64_t z = z0; z < z1; ++z) {
            // one step ahead: the column's plane z + 2 and the halo of plane z + 1
            // (plane z1 is the last one the run reads, the +z neighbour of its last plane)
            const Raw r2 = z + 2 <= z1 ? plane(z + 2) : none;
            Raw h1 = none;
            if (hown && z + 1 < z1) h1 = load(z + 1, hcol, hccol);
            double q0 = 0.0, d0 = 0.0;
            if (MODE == kUpdate && own) {
                q0 = at(A.o1 + z * A.rz, col);
                d0 = at(A.d + z * A.rz, col);
            }
            __syncthreads();  // the previous plane's reads of the tile are done
            sa[ty + 1][tx + 1] = a0;
            sv[ty + 1][tx + 1] = v0;
            if (hr >= 0) {
                sa[hr][hc] = h.a;
                sv[hr][hc] = value(h);
            }
            __syncthreads();
            double res = 0.0;
            if (own) {
                const int r = ty + 1, c = tx + 1;
                const double an[6] = {sa[r][c - 1], sa[r][c + 1], sa[r - 1][c], sa[r + 1][c], am, ap};
                const double vn[6] = {sv[r][c - 1], sv[r][c + 1], sv[r - 1][c], sv[r + 1][c], vm, vp};
                double acc = 0.0;
#pragma unroll
                for (int f = 0; f < 6; ++f) {
                    const double beta = an[f] != 0.0 ? (a0 + fabs(an[f])) * 0.5 : 0.0;
                    const double v = an[f] > 0.0 ? vn[f] : 0.0;
                    acc += beta * (v0 - v);
                }
                double *const o1 = A.o1 + z * A.rz, *const o2 = A.o2 + z * A.rz;
                if (kApply) {
                    const double Lv = a0 > 0.0 ? acc : v0;  // identity row off the fluid
                    put(o1, col, v0);
                    put(o2, col, Lv);
                    dot += v0 * Lv;
                } else if (MODE == kPost) {
                    const double Au = A.scale * acc;
                    const double e = a0 > 0.0 ? v0 + kOmega * s0 * (b0 - Au) : b0;
                    put(o1, col, e);
                    dot += b0 * e;
                } else {
                    res = a0 > 0.0 ? b0 - A.scale * acc : 0.0;
                    if (MODE == kUpdate) {
                        put(o1, col, q0 + coef * d0);
                        put(o2, col, b0);
                        dot += b0 * b0;
                    }
                }
            }
            if (kRestrict) {
                // children (x, y, z): ((c0 + c1) + (c2 + c3)) + ((c4 + c5) + (c6 + c7)),
                // x on the neighbour lane, y 32 lanes on
                double quad = res + __shfl_xor(res, 1);
                quad += __shfl_xor(quad, kTileX);
                if ((z & 1) == 0) half = quad;
                if (((z & 1) || z == nz - 1) && own && ((i | j) & 1) == 0) {
                    const double sum = (z & 1) ? half + quad : half;
                    const int64_t pz = (z >> 1) * A.crz;
                    put(A.bc + pz, ccol, at(A.acc + pz, ccol) > 0.0 ? sum : 0.0);
                }
            }
            am = a0; vm = v0; a0 = ap; v0 = vp; b0 = bp; s0 = sp;
            ap = r2.a; vp = value(r2); bp = rhs(r2); sp = r2.s;
            h = h1;
        }
    }
    if (kApply || MODE == kUpdate || (MODE == kPost && A.part)) {
        dot = block_sum(dot, red);
        const int64_t slot = kApply ? 0 : (MODE == kUpdate ? 2 : 1);
        if (threadIdx.x == 0) A.part[slot * nb + blockIdx.x] = dot;
    }
}

// After the last of a chunk of iterations: its r.r and the stopping test (one
// block), so that the host reads the state of all iterations run.
__global__ void __launch_bounds__(kIdpThreads) k_cg_check(int nb, int k, const double *__restrict__ part,
                                                          CgState *__restrict__ st)
{
    __shared__ double red[kIdpWaves];
    if (st->done >= 0) return;
    const double rr = sum_partials(part + 2 * nb, nb, red);
    if (threadIdx.x == 0) {
        st->rr = rr;
        st->iters = k;
        if (rr <= st->thr) st->done = k;
    }
}

// Iteration k with the Jacobi preconditioner: q += alpha d, r -= alpha w; the
// partials of r.z and r.r.
__global__ void __launch_bounds__(kIdpThreads) k_cg_update(IdpDims D, int k, const double *__restrict__ d,
                                                           const double *__restrict__ w,
                                                           const double *__restrict__ dinv, double *__restrict__ q,
                                                           double *__restrict__ r, double *__restrict__ part,
                                                           const CgState *__restrict__ st)
{
    __shared__ double red[kIdpWaves];
    if (st->done >= 0) return;
    const int nb = gridDim.x;
    const double dw = sum_partials(part, nb, red);
    const double alpha = st->rz[k & 1] / dw;
    double rz = 0.0, rr = 0.0;
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        q[c] += alpha * d[c];
        const double rc = r[c] - alpha * w[c];
        r[c] = rc;
        rz += rc * (rc * dinv[c]);
        rr += rc * rc;
    }
    rz = block_sum(rz, red);
    rr = block_sum(rr, red);
    if (threadIdx.x == 0) {
        part[nb + blockIdx.x] = rz;
        part[2 * nb + blockIdx.x] = rr;
    }
}

// Face displacements (Eq. 13): for the face from cell c to its +axis
// neighbour j, dx (q_c - q_j) with air sides at q = 0, where one side is fluid
// and neither is solid, clamped to [-dx, dx]; faces on the box boundary are
// zero.  The thread of cell c writes the three faces above it and, on the
// lower box faces, the boundary face below it.
__global__ void __launch_bounds__(kIdpThreads) k_idp_faces(IdpDims D, double dx, const double *__restrict__ q,
                                                           const uint8_t *__restrict__ lab, double *__restrict__ fx,
                                                           double *__restrict__ fy, double *__restrict__ fz)
{
#pragma clang fp contract(off)
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        int64_t i, j, k;
        coords(D, c, i, j, k);
        const uint8_t lc = lab[c];
        const double qc = lc == kIdpFluid ? q[c] : 0.0;
        const bool up[3] = {i < D.nx - 1, j < D.ny - 1, k < D.nz - 1};
        const int64_t off[3] = {1, D.nx, D.sxy};
        double *const F[3] = {fx, fy, fz};
        // face index of the face above c along each axis
        const int64_t fi[3] = {(k * D.ny + j) * (D.nx + 1) + i + 1, (k * (D.ny + 1) + j + 1) * D.nx + i,
                               ((k + 1) * D.ny + j) * D.nx + i};
        const int64_t step[3] = {1, D.nx, D.sxy};  // face-index distance to the face below c
        const bool low[3] = {i == 0, j == 0, k == 0};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            double val = 0.0;
            if (up[a]) {
                const uint8_t ln = lab[c + off[a]];
                const bool live =
                    (lc == kIdpFluid || ln == kIdpFluid) && lc != kIdpSolid && ln != kIdpSolid;
                if (live) {
                    const double qn = ln == kIdpFluid ? q[c + off[a]] : 0.0;
                    val = dx * (qc - qn);
                    val = val > -dx ? val : -dx;
                    val = val < dx ? val : dx;
                }
            }
            F[a][fi[a]] = val;
            if (low[a]) F[a][fi[a] - step[a]] = 0.0;
        }
    }
}

// ---------------------------------------------------------------------------
// Multigrid preconditioner: one symmetric V-cycle per CG iteration.  Level
// l + 1 halves level l per axis (rounding up); a coarse cell is air if any of
// its children is air, else fluid if any child is fluid, else solid, and its
// alpha_f' is the mean over its children that are not solid.  The level
// operator is A_l = 4^l L(alpha_f'_l, labels_l), which for constant
// coefficients is the Galerkin product R A_{l-1} P of piecewise-constant
// prolongation P (a fluid coarse cell's correction added to its fluid
// children) and R = P^T (the sum of the fluid children's residuals).
// Smoothing: one damped Jacobi sweep (omega = 2/3) before and one after the
// coarse correction; the pre-sweep from zero, w D^-1 b, is formed on the fly
// where it is used.  A level costs two passes (restriction; correction and
// post-sweep): the finest and levels of at least kMgTiledCells cells blocked
// in 2.5D (k_stencil), the smaller ones a thread per cell; the levels of at
// most kTailTop cells run in one workgroup and one launch (k_mg_tail).
// The coarsest level (at most 256 cells) takes 48 sweeps, as a product with
// their matrix.  Equal pre- and post-sweeps and R = P^T keep the preconditioner
// symmetric.  Non-fluid rows of the finest level are identity rows and get
// z = r.  Levels carry the signed coefficients (see face_sum_ac).
constexpr int kCoarseSweeps = 48;

// uniform per block: read the solver state once
__device__ inline bool cg_done(const CgState *st)
{
    __shared__ int64_t s_done;
    if (threadIdx.x == 0) s_done = st->done;
    __syncthreads();
    return s_done >= 0;
}

__global__ void __launch_bounds__(kIdpThreads) k_mg_coarsen(MgLevel F, MgLevel Cl)
{
    for (int64_t C = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; C < Cl.D.G;
         C += (int64_t)gridDim.x * kIdpThreads) {
        int64_t I, J, K;
        coords(Cl.D, C, I, J, K);
        bool air = false, fluid = false;
        double sum = 0.0;
        int cnt = 0;
        for (int c = 0; c < 2; ++c)
            for (int b = 0; b < 2; ++b)
                for (int a = 0; a < 2; ++a) {
                    const int64_t i = 2 * I + a, j = 2 * J + b, k = 2 * K + c;
                    if (i >= F.D.nx || j >= F.D.ny || k >= F.D.nz) continue;
                    const double v = F.ac[(k * F.D.ny + j) * F.D.nx + i];
                    air |= v < 0.0;
                    fluid |= v > 0.0;
                    if (v != 0.0) {
                        sum += fabs(v);
                        ++cnt;
                    }
                }
        const double mean = cnt ? sum / cnt : 0.0;
        Cl.ac[C] = air ? -mean : (fluid ? mean : 0.0);
    }
}

__global__ void __launch_bounds__(kIdpThreads) k_mg_diag(MgLevel L)
{
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < L.D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        double di = 1.0;
        if (L.ac[c] > 0.0) {
            int64_t i, j, k;
            coords(L.D, c, i, j, k);
            // the face sum of v = 1 on c and 0 on every neighbour is the diagonal
            const double dg =
                face_sum_ac(L.D, c, i, j, k, L.ac, [&](int64_t n, int64_t, int64_t, int64_t) { return n == c ? 1.0 : 0.0; });
            di = dg > 0.0 ? 1.0 / (L.scale * dg) : 0.0;
        }
        L.dinv[c] = di;
    }
}

// Restriction after one pre-smoothing sweep from zero, e1 = w D^-1 b (formed
// on the fly): the coarse right-hand side is the sum of the fluid children's
// residuals b - A e1.  Eight adjacent lanes take the eight children of one
// coarse cell (lane bits: x, y, z offset) and add their residuals with three
// butterfly shuffles, the same order in every group.
__global__ void __launch_bounds__(kIdpThreads) k_mg_restrict(MgLevel F, MgLevel Cl, const CgState *__restrict__ st)
{
    if (cg_done(st)) return;
    auto e1 = [&](int64_t n, int64_t, int64_t, int64_t) { return kOmega * F.dinv[n] * F.b[n]; };
    const int64_t total = 8 * Cl.D.G;  // a multiple of 8: the lanes of a group leave the loop together
    for (int64_t t = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; t < total;
         t += (int64_t)gridDim.x * kIdpThreads) {
        const int64_t C = t >> 3;
        const int ch = (int)(t & 7);
        double v = 0.0;
        if (Cl.ac[C] > 0.0) {
            int64_t I, J, K;
            coords(Cl.D, C, I, J, K);
            const int64_t i = 2 * I + (ch & 1), j = 2 * J + ((ch >> 1) & 1), k = 2 * K + (ch >> 2);
            if (i < F.D.nx && j < F.D.ny && k < F.D.nz) {
                const int64_t f = (k * F.D.ny + j) * F.D.nx + i;
                if (F.ac[f] > 0.0)
                    v = F.b[f] - F.scale * face_sum_ac(F.D, f, i, j, k, F.ac, e1);
            }
        }
        v += __shfl_xor(v, 1);
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 4);
        if (ch == 0) Cl.b[C] = v;
    }
}

// Coarse correction and one post-smoothing sweep: u = e1 + P E, e = u + w D^-1
// (b - A u) (e = b on non-fluid rows).
__global__ void __launch_bounds__(kIdpThreads) k_mg_post(MgLevel F, MgLevel Cl, const CgState *__restrict__ st)
{
    if (cg_done(st)) return;
    auto u = [&](int64_t n, int64_t i, int64_t j, int64_t k) {
        const int64_t p = ((k >> 1) * Cl.D.ny + (j >> 1)) * Cl.D.nx + (i >> 1);
        return kOmega * F.dinv[n] * F.b[n] + Cl.e[p];  // E is zero off the coarse fluid
    };
    for (int64_t c = (int64_t)blockIdx.x * kIdpThreads + threadIdx.x; c < F.D.G;
         c += (int64_t)gridDim.x * kIdpThreads) {
        double z = F.b[c];
        if (F.ac[c] > 0.0) {
            int64_t i, j, k;
            coords(F.D, c, i, j, k);
            const double Au = F.scale * face_sum_ac(F.D, c, i, j, k, F.ac, u);
            z = u(c, i, j, k) + kOmega * F.dinv[c] * (F.b[c] - Au);
        }
        F.e[c] = z;
    }
}

// The operator of the coarsest level's kCoarseSweeps damped Jacobi sweeps from
// zero as a dense matrix, one column per workgroup (the sweeps of a unit
// right-hand side): it depends on the coefficients only, and a product with
// it takes about 1.5 us where the sweeps took 9 to 16 in every cycle.
__global__ void __launch_bounds__(kMgCoarsest) k_mg_coarse_matrix(MgLevel L, double *__restrict__ M)
{
    constexpr int kZero = kMgCoarsest;  // slot that holds zero: neighbours that are no fluid
    __shared__ double sa[kMgCoarsest], se[2][kMgCoarsest + 1];
    const int c = threadIdx.x, n = (int)L.D.G;
    const bool live = c < n;
    sa[c] = live ? L.ac[c] : 0.0;
    se[0][c] = 0.0;
    if (c < 2) se[c][kZero] = 0.0;
    __syncthreads();
    const double a = sa[c];
    double beta[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, di = 0.0;
    int slot[6] = {kZero, kZero, kZero, kZero, kZero, kZero};
    if (a > 0.0) {
        int64_t i, j, k;
        coords(L.D, c, i, j, k);
        Nbr nb[6];
        neighbours(L.D, i, j, k, nb);
        di = L.dinv[c];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const double an = nb[f].inside ? sa[c + nb[f].off] : 0.0;
            beta[f] = an != 0.0 ? (a + fabs(an)) * 0.5 : 0.0;
            if (an > 0.0) slot[f] = (int)(c + nb[f].off);
        }
    }
    const double b = c == (int)blockIdx.x ? 1.0 : 0.0;
    double v = 0.0;
    for (int s = 0; s < kCoarseSweeps; ++s) {
        const int cur = s & 1;
        if (a > 0.0) {
            double acc = 0.0;
#pragma unroll
            for (int f = 0; f < 6; ++f) acc += beta[f] * (v - se[cur][slot[f]]);
            v = v + kOmega * di * (b - L.scale * acc);
        }
        if (live) se[cur ^ 1][c] = v;
        __syncthreads();
    }
    if (live) M[(int64_t)blockIdx.x * n + c] = v;
}

// The V-cycle's small levels in one workgroup and one launch: the first of at
// most kTailTop cells, all below it of at most one cell per thread.  Their
// coefficients and values are held in LDS, the first level's right-hand side
// and 1 / diag in registers, so that between the first loads and the last
// stores there are only LDS passes and barriers: restriction (residual, then
// the sums of the children in k_mg_restrict's order), the coarsest matrix,
// correction and sweep (k_mg_post).  Levels of 1,024 and 128 cells take 10.8
// us, 4,096 to 64 cells 15.6; the same levels in launches of their own took
// 4.5 to 5.2 us a pass and the coarsest sweeps 17.
constexpr int kTailThreads = 1024;
constexpr int kTailTop = 4096, kTailBelow = 2048;  // cells of the first level and of all below
constexpr int kTailCells = kTailTop / kTailThreads;
constexpr int kTailLevels = 8;

struct MgTail {
    int n;
    MgLevel lev[kTailLevels];
    const double *M;  // the coarsest level's matrix
};

__global__ void __launch_bounds__(kTailThreads) k_mg_tail(MgTail T, const CgState *__restrict__ st)
{
    __shared__ double sa[kTailTop + kTailBelow], sv[kTailTop + kTailBelow], sb[kTailBelow], sd[kTailBelow];
    if (cg_done(st)) return;
    const int tid = threadIdx.x;
    const MgLevel &F0 = T.lev[0];
    const int G0 = (int)F0.D.G;
    double b0[kTailCells], d0[kTailCells];
#pragma unroll
    for (int u = 0; u < kTailCells; ++u) {
        const int c = tid + u * kTailThreads;
        b0[u] = d0[u] = 0.0;
        if (c < G0) {
            b0[u] = F0.b[c];
            d0[u] = F0.dinv[c];
            sa[c] = F0.ac[c];
            sv[c] = kOmega * d0[u] * b0[u];
        }
    }
    int below = 0;  // first slot of level l in sb, sd; level l > 0 has kTailTop + below in sa, sv
    for (int l = 1; l < T.n; ++l) {
        const int G = (int)T.lev[l].D.G;
        if (tid < G) {
            sa[kTailTop + below + tid] = T.lev[l].ac[tid];
            sd[below + tid] = T.lev[l].dinv[tid];
        }
        below += G;
    }
    __syncthreads();
    // residual of the cell c after the pre-sweep, or the post-sweep's result
    auto face = [&](const MgLevel &L, int base, int c) {
        int64_t i, j, k;
        coords(L.D, c, i, j, k);
        return L.scale * face_sum_ac(L.D, (int64_t)c, i, j, k, sa + base,
                                     [&](int64_t n, int64_t, int64_t, int64_t) { return sv[base + n]; });
    };
    int at = 0, off = 0;  // this level's slots in sa, sv and in sb, sd
    for (int l = 0; l + 1 < T.n; ++l) {
        const MgLevel &F = T.lev[l], &C = T.lev[l + 1];
        const int G = (int)F.D.G, cat = l == 0 ? kTailTop : at + G, coff = l == 0 ? 0 : off + G;
        double r[kTailCells];
#pragma unroll
        for (int u = 0; u < kTailCells; ++u) {
            const int c = tid + u * kTailThreads;
            r[u] = 0.0;
            if (c < G && sa[at + c] > 0.0) r[u] = (l == 0 ? b0[u] : sb[off + c]) - face(F, at, c);
            if (l > 0) break;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTailCells; ++u) {
            const int c = tid + u * kTailThreads;
            if (c < G) sv[at + c] = r[u];
            if (l > 0) break;
        }
        __syncthreads();
        if (tid < (int)C.D.G) {
            int64_t I, J, K;
            coords(C.D, tid, I, J, K);
            double c[8];
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const int64_t i = 2 * I + (ch & 1), j = 2 * J + ((ch >> 1) & 1), k = 2 * K + (ch >> 2);
                c[ch] = i < F.D.nx && j < F.D.ny && k < F.D.nz ? sv[at + (k * F.D.ny + j) * F.D.nx + i] : 0.0;
            }
            const double sum = ((c[0] + c[1]) + (c[2] + c[3])) + ((c[4] + c[5]) + (c[6] + c[7]));
            const double b = sa[cat + tid] > 0.0 ? sum : 0.0;
            sb[coff + tid] = b;
            sv[cat + tid] = kOmega * sd[coff + tid] * b;
        }
        __syncthreads();
        at = cat;
        off = coff;
    }
    {  // the coarsest level: its matrix times b, the columns shared by the waves
        const int n = (int)T.lev[T.n - 1].D.G;
        if (T.n == 1) {
            if (tid < n) sb[tid] = b0[0];
            __syncthreads();
        }
        const int pad = n <= 64 ? 64 : (n <= 128 ? 128 : 256), parts = kTailThreads / pad;
        const int c = tid & (pad - 1), p = tid / pad, per = (n + parts - 1) / parts;
        double sum = 0.0;
        if (c < n) {
            const int j1 = (p + 1) * per < n ? (p + 1) * per : n;
#pragma unroll 4
            for (int j = p * per; j < j1; ++j) sum += T.M[(int64_t)j * n + c] * sb[off + j];
        }
        // the partial sums take the first level's last coefficient slots for a
        // moment (nothing reads them here; they are put back)
        __syncthreads();
        double *part = sa + kTailTop - kTailThreads;
        const double keep = part[tid];
        part[tid] = sum;
        __syncthreads();
        double e = 0.0;
        if (tid < n) {
            for (int q = 0; q < parts; ++q) e += part[q * pad + tid];
            sv[at + tid] = e;
        }
        __syncthreads();
        part[tid] = keep;
        if (T.n == 1 && tid < n) T.lev[0].e[tid] = e;
        __syncthreads();
    }
    for (int l = T.n - 2; l >= 0; --l) {
        const MgLevel &F = T.lev[l], &C = T.lev[l + 1];
        const int G = (int)F.D.G, cat = at;
        at = l == 0 ? 0 : cat - G;
        off = l == 0 ? 0 : off - G;
        double e[kTailCells];
#pragma unroll
        for (int u = 0; u < kTailCells; ++u) {
            const int c = tid + u * kTailThreads;
            if (c < G) {
                int64_t i, j, k;
                coords(F.D, c, i, j, k);
                const int64_t p = ((k >> 1) * C.D.ny + (j >> 1)) * C.D.nx + (i >> 1);
                sv[at + c] = kOmega * (l == 0 ? d0[u] : sd[off + c]) * (l == 0 ? b0[u] : sb[off + c]) + sv[cat + p];
            }
            if (l > 0) break;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTailCells; ++u) {
            const int c = tid + u * kTailThreads;
            const double b = l == 0 ? b0[u] : (c < G ? sb[off + c] : 0.0);
            e[u] = b;
            if (c < G && sa[at + c] > 0.0)
                e[u] = sv[at + c] + kOmega * (l == 0 ? d0[u] : sd[off + c]) * (b - face(F, at, c));
            if (l > 0) break;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTailCells; ++u) {
            const int c = tid + u * kTailThreads;
            if (c < G) {
                if (l == 0)
                    F.e[c] = e[u];
                else
                    sv[at + c] = e[u];
            }
            if (l > 0) break;
        }
        __syncthreads();
    }
}

unsigned idp_blocks(int64_t G)
{
    const int64_t b = (G + 127) / 128;  // small grids: short runs of planes in more blocks
    return (unsigned)(b < 1 ? 1 : (b > kIdpMaxBlocks ? kIdpMaxBlocks : b));
}

// One thread per cell for kernels that write no partials (grid-stride
// beyond 2^31 - 1 blocks).
unsigned idp_blocks_full(int64_t G)
{
    const int64_t b = (G + kIdpThreads - 1) / kIdpThreads;
    return (unsigned)(b < 1 ? 1 : (b > 0x7fffffffll ? 0x7fffffffll : b));
}

}  // namespace

// m = ceil(2^(31+s) / d) with 2^(s-1) < d <= 2^s: m < 2^32, and m d - 2^(31+s)
// < d <= 2^s, so floor(n m / 2^(31+s)) = floor(n / d) for every n < 2^31
// (the round-up reciprocal of Granlund and Montgomery, 1994).
static void div_constants(int64_t d, uint32_t &m, int32_t &sh)
{
    int s = 0;
    while ((int64_t(1) << s) < d) ++s;
    if (d < 1 || s > 31) {  // grids of 2^31 cells or more divide in 64 bits
        m = 0;
        sh = 0;
        return;
    }
    m = (uint32_t)(((uint64_t(1) << (31 + s)) + (uint64_t)d - 1) / (uint64_t)d);
    sh = 31 + s;
}

void idp_dims_finish(IdpDims &D)
{
    D.sxy = D.nx * D.ny;
    D.G = D.sxy * D.nz;
    div_constants(D.nx, D.mx, D.shx);
    div_constants(D.ny, D.my, D.shy);
}

IdpDims idp_dims(const DevParams &P)
{
    IdpDims D;
    D.nx = P.n[0];
    D.ny = P.n[1];
    D.nz = P.n[2];
    idp_dims_finish(D);
    return D;
}

// Axes of one cell hold no faces between cells, so the solver takes the others for
// x, y and z: the cells lie in the same order, and a face sum and a coarse cell's
// children add the same terms in the same order.  Flat grids then fill the tiles
// of the stencil passes, and columns their rows (512 x 1 x 512 cells, Jacobi 58.7
// -> 37.0 ms, multigrid 32.0 -> 21.9; 1 x 1 x 32,767, multigrid 619 -> 159).
IdpDims idp_solve_dims(const DevParams &P)
{
    int64_t d[3] = {1, 1, 1};
    int k = 0;
    for (int a = 0; a < 3; ++a)
        if (P.n[a] > 1) d[k++] = P.n[a];
    IdpDims D;
    D.nx = d[0];
    D.ny = d[1];
    D.nz = d[2];
    idp_dims_finish(D);
    return D;
}

hipError_t launch_idp_setup(const IdpDims &D, double alpha_max, const int64_t *afx, const double *astar,
                            const uint8_t *lab, double *at, double *s, int64_t *err, hipStream_t st)
{
    k_idp_setup<<<idp_blocks(D.G), kIdpThreads, 0, st>>>(D, alpha_max, afx, astar, lab, at, s, err);
    return hipGetLastError();
}

hipError_t launch_idp_apply(const IdpDims &D, const double *at, const uint8_t *lab, const double *v, double *out,
                            hipStream_t st)
{
    k_idp_apply<<<idp_blocks(D.G), kIdpThreads, 0, st>>>(D, at, lab, v, out);
    return hipGetLastError();
}

hipError_t launch_idp_faces(const IdpDims &D, double dx, const double *q, const uint8_t *lab, double *fx,
                            double *fy, double *fz, hipStream_t st)
{
    k_idp_faces<<<idp_blocks(D.G), kIdpThreads, 0, st>>>(D, dx, q, lab, fx, fy, fz);
    return hipGetLastError();
}

// Levels with at least this many cells take the passes blocked in 2.5D (the
// finest always does); on smaller ones a thread per cell is faster, the grid
// being too small for runs of planes.
constexpr int64_t kMgTiledCells = 1 << 18;

// Axes of a blocked stencil pass over D: with fewer rows than half a tile's and
// more planes, the tiles lie in x and z and the runs go along y, so that the tiles
// are full and the runs short (1,024 x 4 x 1,024 cells, multigrid 140 -> 84 ms,
// Jacobi 197 -> 155; at 8 rows no difference with 256 planes, 12 % slower with 300
// planes of 8 x 8).
// Then its tiles, and the planes per item (even, so that a coarse cell's children
// lie in one run): about one item per block of nb.
static void stencil_items(const IdpDims &D, unsigned nb, StencilArgs &A)
{
    A.exchanged = 2 * D.ny < kTileY && D.nz > D.ny;
    A.nx = D.nx;
    A.ny = A.exchanged ? D.nz : D.ny;
    A.nz = A.exchanged ? D.ny : D.nz;
    A.ry = A.exchanged ? D.sxy : D.nx;
    A.rz = A.exchanged ? D.nx : D.sxy;
    A.ntx = (int)((A.nx + kTileX - 1) / kTileX);
    A.nty = (int)((A.ny + kTileY - 1) / kTileY);
    int64_t zl = (A.nz * A.ntx * A.nty + nb - 1) / nb;
    zl = (zl + 1) / 2 * 2;
    A.zlen = (int)(zl > A.nz + 1 ? A.nz + 1 : zl);
    if (A.zlen & 1) ++A.zlen;
}

static void stencil_coarse(const IdpDims &C, StencilArgs &A)
{
    A.cry = A.exchanged ? C.sxy : C.nx;
    A.crz = A.exchanged ? C.nx : C.sxy;
}

template <int MODE>
static void launch_stencil(const StencilArgs &A, unsigned nb, hipStream_t st)
{
    if (A.ny * A.ry < (int64_t)1 << 29)
        k_stencil<MODE, uint32_t><<<nb, kIdpThreads, 0, st>>>(A);
    else
        k_stencil<MODE, uint64_t><<<nb, kIdpThreads, 0, st>>>(A);
}

static StencilArgs stencil_args(const IdpDims &D, const IdpWork &W, unsigned nb)
{
    StencilArgs A;
    memset(&A, 0, sizeof(A));
    stencil_items(D, nb, A);
    A.scale = 1.0;
    A.ac = W.lev[0].ac;
    A.dinv = W.dinv;
    A.part = W.part;
    A.st = W.state;
    return A;
}

// The finest level's r and z and the directions live in two buffers each that
// change places every iteration (see k_stencil): r of iteration k in
// rbuf(k), z in rbuf(k + 1), d in dbuf(k).
static double *rbuf(const IdpWork &W, int k) { return (k & 1) ? W.lev[0].e : W.r; }
static double *dbuf(const IdpWork &W, int k) { return (k & 1) ? W.lev[0].t : W.d; }

static void residual_pass(const MgLevel &F, const MgLevel &C, const double *b, const IdpWork &W, hipStream_t st)
{
    const unsigned nb = idp_blocks(F.D.G);
    StencilArgs A = stencil_args(F.D, W, nb);
    A.scale = F.scale;
    A.ac = F.ac;
    A.dinv = F.dinv;
    A.p = b;
    A.acc = C.ac;
    stencil_coarse(C.D, A);
    A.bc = C.b;
    launch_stencil<kResidual>(A, nb, st);
}

static void post_pass(const MgLevel &F, const MgLevel &C, const double *b, double *e, double *part, const IdpWork &W,
                      hipStream_t st)
{
    const unsigned nb = idp_blocks(F.D.G);
    StencilArgs A = stencil_args(F.D, W, nb);
    A.scale = F.scale;
    A.ac = F.ac;
    A.dinv = F.dinv;
    A.p = b;
    A.ec = C.e;
    stencil_coarse(C.D, A);
    A.o1 = e;
    A.part = part;
    launch_stencil<kPost>(A, nb, st);
}

// The V-cycle below the finest level: from level 1's right-hand side to its
// correction.
static void launch_coarse(const IdpWork &W, hipStream_t st)
{
    // the first level that, with all below it, fits one workgroup
    auto fits = [&](int l) {
        int64_t below = 0;
        for (int m = l + 1; m < W.nlev; ++m) {
            if (W.lev[m].D.G > kTailThreads) return false;
            below += W.lev[m].D.G;
        }
        return W.lev[l].D.G <= kTailTop && below <= kTailBelow && W.nlev - l <= kTailLevels;
    };
    int tail = 1;
    while (!fits(tail)) ++tail;
    for (int l = 1; l < tail; ++l) {
        const MgLevel &F = W.lev[l], &C = W.lev[l + 1];
        if (F.D.G >= kMgTiledCells)
            residual_pass(F, C, F.b, W, st);
        else
            k_mg_restrict<<<idp_blocks_full(8 * C.D.G), kIdpThreads, 0, st>>>(F, C, W.state);
    }
    MgTail T;
    T.n = W.nlev - tail;
    for (int l = 0; l < T.n; ++l) T.lev[l] = W.lev[tail + l];
    T.M = W.coarse;
    k_mg_tail<<<1, kTailThreads, 0, st>>>(T, W.state);
    for (int l = tail - 1; l >= 1; --l) {
        const MgLevel &F = W.lev[l], &C = W.lev[l + 1];
        if (F.D.G >= kMgTiledCells)
            post_pass(F, C, F.b, F.e, nullptr, W, st);
        else
            k_mg_post<<<idp_blocks(F.D.G), kIdpThreads, 0, st>>>(F, C, W.state);
    }
}

hipError_t launch_cg_start(const IdpDims &D, const double *at, const uint8_t *lab, const double *s, const double *q,
                           const IdpWork &W, double tol, int64_t *err, hipStream_t st)
{
    const unsigned nb = idp_blocks(D.G);
    k_cg_init<<<nb, kIdpThreads, 0, st>>>(D, at, lab, s, q, W.r, W.dinv, W.lev[0].ac, W.part, W.state, err);
    if (W.nlev > 1) {
        for (int l = 0; l + 1 < W.nlev; ++l) {
            k_mg_coarsen<<<idp_blocks(W.lev[l + 1].D.G), kIdpThreads, 0, st>>>(W.lev[l], W.lev[l + 1]);
            k_mg_diag<<<idp_blocks(W.lev[l + 1].D.G), kIdpThreads, 0, st>>>(W.lev[l + 1]);
        }
        const MgLevel &L = W.lev[W.nlev - 1];
        k_mg_coarse_matrix<<<(unsigned)L.D.G, (unsigned)kMgCoarsest, 0, st>>>(L, W.coarse);
        residual_pass(W.lev[0], W.lev[1], rbuf(W, 0), W, st);
        launch_coarse(W, st);
        post_pass(W.lev[0], W.lev[1], rbuf(W, 0), rbuf(W, 1), W.part, W, st);
    }
    k_cg_start<<<1, kIdpThreads, 0, st>>>((int)nb, W.part, tol, W.state);
    return hipGetLastError();
}

hipError_t launch_cg_iterations(const IdpDims &D, const double *at, const uint8_t *lab, double *q,
                                const IdpWork &W, int k0, int count, hipStream_t st)
{
    const unsigned nb = idp_blocks(D.G);
    const bool mg = W.nlev > 1;
    for (int k = k0; k < k0 + count; ++k) {
        StencilArgs A = stencil_args(D, W, nb);
        A.k = k;
        A.d = dbuf(W, k + 1);
        A.o1 = dbuf(W, k);
        A.o2 = W.w;
        A.p = mg ? rbuf(W, k + 1) : W.r;
        if (!mg) {
            launch_stencil<kApplyJac>(A, nb, st);
            k_cg_update<<<nb, kIdpThreads, 0, st>>>(D, k, dbuf(W, k), W.w, W.dinv, q, W.r, W.part, W.state);
            continue;
        }
        launch_stencil<kApplyMg>(A, nb, st);
        A.p = rbuf(W, k);
        A.d = dbuf(W, k);
        A.w = W.w;
        A.acc = W.lev[1].ac;
        stencil_coarse(W.lev[1].D, A);
        A.bc = W.lev[1].b;
        A.o1 = q;
        A.o2 = rbuf(W, k + 1);
        launch_stencil<kUpdate>(A, nb, st);
        launch_coarse(W, st);
        post_pass(W.lev[0], W.lev[1], rbuf(W, k + 1), rbuf(W, k + 2), W.part, W, st);
    }
    k_cg_check<<<1, kIdpThreads, 0, st>>>((int)nb, k0 + count, W.part, W.state);
    return hipGetLastError();
}

}  // namespace gic
