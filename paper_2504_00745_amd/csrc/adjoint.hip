// a9: adjoint (vector-Jacobian products) of the granule step on gfx950, in
// double.  Forward definitions (Sec. 3.1 Eq. 1a-c; Sec. 3.3 Eq. 5b with the
// App. A relaxation drag; Sec. 5.1 Eq. 7a; Sec. 5.2 G2P; Sec. 4 symplectic
// Euler), unquantised transfers:
//   A = P2G_alpha(x);  (u_at, alpha_f) = G2P(x; u, A);
//   F_d = C_d 6 pi eta r alpha_f (u_at - v);  F_c = contact(x, v; mu);
//   v' = v + dt ((F_c + F_d)/m + g);  x' = x + dt v'.
// Every kernel reads its forward inputs and recomputes what it needs; the
// contact pullback (contact.hip) is a gather (granule i collects, for each
// touching partner j, the pair term with cotangent g_i - g_j), so no atomics
// are used except in the grid scatter of the G2P pullback, which sums integers
// (contributions rounded at the scale of the largest one; transfer.hip), so
// every result is the same bits in every run.
//
// The rollout's step and its reverse (gic_rollout_step, gic_rollout_step_vjp)
// run in eight and ten launches (more where their sort passes over digits, or the
// contact pulls run by granule): on beds of 65,536 granules a launch costs 3
// to 5 us whatever it does, and the separate stages were 17 and 28 of them,
// each reading the bed again.  Loss and gradients of 20 steps of that bed, as
// a replayed graph: 10.07 -> 5.39 ms; of 6 steps of 4,096 granules launched
// one by one: 4.19 -> 1.35 ms.
#include "gic_launch.hpp"

namespace gic {

namespace {

__global__ void __launch_bounds__(256) k_drag_vjp(DevParams P, int64_t n, const double *__restrict__ r,
                                                  const double *__restrict__ v, const double *__restrict__ uat,
                                                  const double *__restrict__ af, const double *__restrict__ gF,
                                                  double *__restrict__ gv, double *__restrict__ guat,
                                                  double *__restrict__ gaf, double *__restrict__ gcd)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const double c = P.cdrag_unit * r[q];   // 6 pi eta r
    const double beta = P.c_drag * c;
    double s = 0.0;
    for (int a = 0; a < 3; ++a) {
        const double g = gF[a * n + q];
        gv[a * n + q] += -beta * af[q] * g;
        guat[a * n + q] = beta * af[q] * g;
        s += (uat[a * n + q] - v[a * n + q]) * g;
    }
    gaf[q] = beta * s;
    gcd[q] = c * af[q] * s;
}

// dL/dx^{n+1} = gx, dL/dv^{n+1} = gv on entry.  v^{n+1} feeds x^{n+1}, so
// its total adjoint is gv + dt gx (written back to gv: this is also the
// adjoint of v^n through the identity term); gF = dt/m of it.
__global__ void __launch_bounds__(256) k_integrate_vjp(DevParams P, int64_t n, const double *__restrict__ r,
                                                       const double *__restrict__ gx, double *__restrict__ gv,
                                                       double *__restrict__ gF)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const double s = P.dt / mass_of(P, r[q]);
    for (int a = 0; a < 3; ++a) {
        const double t = gv[a * n + q] + P.dt * gx[a * n + q];
        gv[a * n + q] = t;
        gF[a * n + q] = s * t;
    }
}

// Granule part of the G2P pullback: gx += sum_k grad w_k (u_k . guat -
// min(A_k, alpha_max) gaf).
__global__ void __launch_bounds__(256) k_g2p_vjp_x(DevParams P, int64_t n, const double *__restrict__ x,
                                                   const double *__restrict__ u, const double *__restrict__ A,
                                                   const double *__restrict__ guat, const double *__restrict__ gaf,
                                                   double *__restrict__ gx)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const double xa[3] = {x[q], x[n + q], x[2 * n + q]};
    Stencil s;
    stencil_of(P, xa, s);
    double dw[3][3];
    stencil_dw(P, xa, dw);
    const int64_t G = P.G;
    const double gu[3] = {guat[q], guat[n + q], guat[2 * n + q]};
    const double ga = gaf[q];
    double acc[3] = {0, 0, 0};
    for (int cz = 0; cz < 3; ++cz)
        for (int cy = 0; cy < 3; ++cy)
            for (int cx = 0; cx < 3; ++cx) {
                const int64_t k = node_index(P, s.node[0][cx], s.node[1][cy], s.node[2][cz]);
                const double ul = (u[k] * gu[0] + u[G + k] * gu[1]) + u[2 * G + k] * gu[2];
                const double al = A[k] < P.alpha_max ? A[k] : P.alpha_max;
                const double coef = ul - al * ga;
                acc[0] += (dw[0][cx] * s.w[1][cy]) * s.w[2][cz] * coef;
                acc[1] += (s.w[0][cx] * dw[1][cy]) * s.w[2][cz] * coef;
                acc[2] += (s.w[0][cx] * s.w[1][cy]) * dw[2][cz] * coef;
            }
    for (int a = 0; a < 3; ++a) gx[a * n + q] += acc[a];
}

// P2G pullback (gather): gx += frac sum_k gA_k grad w_k + m sum_k (gP_k . v)
// grad w_k;  gv += m sum_k w_k gP_k.
__global__ void __launch_bounds__(256) k_p2g_vjp(DevParams P, int64_t n, const double *__restrict__ x,
                                                 const double *__restrict__ v, const double *__restrict__ r,
                                                 const double *__restrict__ gA, const double *__restrict__ gP,
                                                 double *__restrict__ gx, double *__restrict__ gv)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const double xa[3] = {x[q], x[n + q], x[2 * n + q]};
    Stencil s;
    stencil_of(P, xa, s);
    double dw[3][3];
    stencil_dw(P, xa, dw);
    const int64_t G = P.G;
    const double frac = volume_of(r[q]) * P.inv_vcell;
    const double m = mass_of(P, r[q]);
    const double vq[3] = {v[q], v[n + q], v[2 * n + q]};
    double ax[3] = {0, 0, 0}, av[3] = {0, 0, 0};
    for (int cz = 0; cz < 3; ++cz)
        for (int cy = 0; cy < 3; ++cy)
            for (int cx = 0; cx < 3; ++cx) {
                const int64_t k = node_index(P, s.node[0][cx], s.node[1][cy], s.node[2][cz]);
                const double w = (s.w[0][cx] * s.w[1][cy]) * s.w[2][cz];
                double coef = 0.0;
                if (gA) coef += gA[k] * frac;
                if (gP) {
                    const double g3[3] = {gP[k], gP[G + k], gP[2 * G + k]};
                    coef += m * ((g3[0] * vq[0] + g3[1] * vq[1]) + g3[2] * vq[2]);
                    for (int a = 0; a < 3; ++a) av[a] += m * w * g3[a];
                }
                ax[0] += (dw[0][cx] * s.w[1][cy]) * s.w[2][cz] * coef;
                ax[1] += (s.w[0][cx] * dw[1][cy]) * s.w[2][cz] * coef;
                ax[2] += (s.w[0][cx] * s.w[1][cy]) * dw[2][cz] * coef;
            }
    for (int a = 0; a < 3; ++a) {
        gx[a * n + q] += ax[a];
        gv[a * n + q] += av[a];
    }
}

// Deterministic sum: fixed per-workgroup partial sums (wave shuffles, then
// LDS), then one workgroup adds the partials in index order.
__global__ void __launch_bounds__(256) k_partial_sums(const double *__restrict__ a, const double *__restrict__ b,
                                                      int64_t n, int64_t per, double *__restrict__ part)
{
    __shared__ double w[4];
    const int64_t lo = (int64_t)blockIdx.x * per;
    const int64_t hi = lo + per < n ? lo + per : n;
    double s = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 256) s += b ? a[i] * b[i] : a[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = ((w[0] + w[1]) + w[2]) + w[3];
}

__global__ void __launch_bounds__(256) k_final_sum(const double *__restrict__ part, int nb, double *out, int acc)
{
    __shared__ double w[4];
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256) s += part[i];
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double t = ((w[0] + w[1]) + w[2]) + w[3];
        *out = acc ? *out + t : t;
    }
}

// out = (factor s[0]) a, s a device scalar (a cotangent that stays on the
// device).
__global__ void __launch_bounds__(256) k_scale(int64_t n, const double *__restrict__ a, const double *__restrict__ sp,
                                               double factor, double *__restrict__ out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    out[i] = (factor * sp[0]) * a[i];
}

__global__ void __launch_bounds__(256) k_permute(int64_t n, int comps, const int32_t *__restrict__ order,
                                                 const double *__restrict__ in, double *__restrict__ out, int scatter)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= n) return;
    const int64_t i = order[q];
    if ((uint64_t)i >= (uint64_t)n) return;  // not a permutation of [0, n): left untouched
    for (int c = 0; c < comps; ++c) {
        if (scatter)
            out[c * n + i] = in[c * n + q];
        else
            out[c * n + q] = in[c * n + i];
    }
}

}  // namespace

hipError_t launch_drag_vjp(const DevParams &P, int64_t n, const double *r, const double *v, const double *uat,
                           const double *af, const double *gF, double *gv, double *guat, double *gaf, double *gcd,
                           hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_drag_vjp<<<grid_for(n, 256), 256, 0, s>>>(P, n, r, v, uat, af, gF, gv, guat, gaf, gcd);
    return hipGetLastError();
}

hipError_t launch_integrate_vjp(const DevParams &P, int64_t n, const double *r, const double *gx, double *gv,
                                double *gF, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_integrate_vjp<<<grid_for(n, 256), 256, 0, s>>>(P, n, r, gx, gv, gF);
    return hipGetLastError();
}

hipError_t launch_g2p_vjp(const DevParams &P, int64_t n, int64_t K, const double *x, const double *u,
                          const double *A, const double *guat, const double *gaf, const int32_t *cb,
                          const int32_t *ce, const BrickList &B, double *gx, double *gA, int64_t *fx, double *part,
                          hipStream_t s)
{
    if (n > 0) k_g2p_vjp_x<<<grid_for(n, 256), 256, 0, s>>>(P, n, x, u, A, guat, gaf, gx);
    if (gA) return launch_g2p_vjp_grid(P, n, K, x, A, gaf, cb, ce, B, gA, fx, part, s);
    return hipGetLastError();
}

hipError_t launch_p2g_vjp(const DevParams &P, int64_t n, const double *x, const double *v, const double *r,
                          const double *gA, const double *gP, double *gx, double *gv, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_p2g_vjp<<<grid_for(n, 256), 256, 0, s>>>(P, n, x, v, r, gA, gP, gx, gv);
    return hipGetLastError();
}

hipError_t launch_sum(const double *a, const double *b, int64_t n, double *part, int nparts, double *out, int acc,
                      hipStream_t s)
{
    const int64_t per = n > 0 ? (n + nparts - 1) / nparts : 1;
    const int nb = (int)(n > 0 ? (n + per - 1) / per : 0);
    if (nb > 0) k_partial_sums<<<nb, 256, 0, s>>>(a, b, n, per, part);
    k_final_sum<<<1, 256, 0, s>>>(part, nb, out, acc);
    return hipGetLastError();
}

namespace {

// Last pass of a reverse step: the P2G pullback of g_alpha (held as integer
// sums fx2 at the scale of the largest |g_alpha_f| bits), and the adjoint of
// (x, v) back in input order.  The first workgroup adds the bricks' (or
// workgroups') partial sums of dL/dmu and dL/dC_d to the scalars, in their order.
__global__ void __launch_bounds__(256) k_rollout_pull(DevParams P, int64_t n, const int32_t *__restrict__ order,
                                                      const double *__restrict__ x, const double *__restrict__ r,
                                                      const int64_t *__restrict__ fx2,
                                                      const unsigned long long *__restrict__ gmax,
                                                      const double *__restrict__ gs, double *__restrict__ gxv,
                                                      const double *__restrict__ psum, const int32_t *__restrict__ count,
                                                      int parts,
                                                      double *__restrict__ gmu, double *__restrict__ gcd)
{
    if (blockIdx.x == 0) {
        __shared__ double w[2][4];
        double m = 0.0, c = 0.0;
        int np = parts;  // per workgroup of granules or per brick, see launch_rollout_contact
        if (np < 0) np = pull_granules(n, *count) ? -np : 0;
        if (np == 0) np = *count;
        for (int i = threadIdx.x; i < np; i += 256) {
            m += psum[2 * i];
            c += psum[2 * i + 1];
        }
        for (int off = 32; off > 0; off >>= 1) {
            m += __shfl_xor(m, off);
            c += __shfl_xor(c, off);
        }
        if ((threadIdx.x & 63) == 0) {
            w[0][threadIdx.x >> 6] = m;
            w[1][threadIdx.x >> 6] = c;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            *gmu += ((w[0][0] + w[0][1]) + w[0][2]) + w[0][3];
            *gcd += ((w[1][0] + w[1][1]) + w[1][2]) + w[1][3];
        }
    }
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= n) return;
    const int64_t i = order[q];
    const double inv = 1.0 / fix_scale(__longlong_as_double((long long)*gmax));
    const double xa[3] = {x[q], x[n + q], x[2 * n + q]};
    Stencil s;
    stencil_of(P, xa, s);
    double dw[3][3];
    stencil_dw(P, xa, dw);
    const double frac = volume_of(r[q]) * P.inv_vcell;
    double ax[3] = {0, 0, 0};
    for (int cz = 0; cz < 3; ++cz)
        for (int cy = 0; cy < 3; ++cy)
            for (int cx = 0; cx < 3; ++cx) {
                const int64_t k = node_index(P, s.node[0][cx], s.node[1][cy], s.node[2][cz]);
                const double coef = ((double)fx2[k] * inv) * frac;
                ax[0] += (dw[0][cx] * s.w[1][cy]) * s.w[2][cz] * coef;
                ax[1] += (s.w[0][cx] * dw[1][cy]) * s.w[2][cz] * coef;
                ax[2] += (s.w[0][cx] * s.w[1][cy]) * dw[2][cz] * coef;
            }
    if ((uint64_t)i >= (uint64_t)n) return;
    for (int a = 0; a < 3; ++a) {
        gxv[a * n + i] = gs[a * n + q] + ax[a];
        gxv[(3 + a) * n + i] = gs[(3 + a) * n + q];
    }
}

}  // namespace

hipError_t launch_rollout_pull(const DevParams &P, int64_t n, const int32_t *order, const double *x, const double *r,
                               const int64_t *fx2, const unsigned long long *gmax, const double *gs, double *gxv,
                               const double *psum, const BrickList &B, int parts, double *gmu, double *gcd, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_rollout_pull<<<grid_for(n, 256), 256, 0, s>>>(P, n, order, x, r, fx2, gmax, gs, gxv, psum, B.count, parts, gmu,
                                                    gcd);
    return hipGetLastError();
}

hipError_t launch_scale(int64_t n, const double *a, const double *sp, double factor, double *out, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_scale<<<grid_for(n, 256), 256, 0, s>>>(n, a, sp, factor, out);
    return hipGetLastError();
}

hipError_t launch_permute(int64_t n, int comps, const int32_t *order, const double *in, double *out, int scatter,
                          hipStream_t s)
{
    if (n == 0) return hipSuccess;
    k_permute<<<grid_for(n, 256), 256, 0, s>>>(n, comps, order, in, out, scatter);
    return hipGetLastError();
}

}  // namespace gic
