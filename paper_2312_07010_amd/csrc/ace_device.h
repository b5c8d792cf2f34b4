// Device-side building blocks of the RLB-MIE-FD step for gfx950 (wave64).
//
// The step (Sec. 2, pointwise form IE-FD) at a node with value p is
//   xi    = p + kappa * sum_k (p_{+k} + p_{-k} - 2 p) - h (p^3 - p),
//   p_new = the unique real root theta of theta + h (theta^3 - theta) = xi
// (Sec. 3.2, Remark 1: unique for 0 < dt < 2), with h = dt/2.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ace_internal.h"

namespace ace {

// Unique real root theta of theta + h (theta^3 - theta) = xi, 0 < h < 1.
//
// For |xi| <= 1 (always the case under Theorem 2's conditions) and dt up to
// 0.05 the root is the polynomial theta = xi + xi w S(w), w = 1 - xi^2:
// (theta - xi) / (xi w) is an analytic function of w on [0, 1], which the
// host interpolates with the least degree of ROOT_DEG that brings theta
// within 2^-60 of the root (choose_root in ace_api.hip).  It takes
// deg + 3 instructions (6 at dt = 5e-4, 7 at 1e-3), where a Newton step from
// an expansion of the root takes 12, one of them a quarter-rate reciprocal.
// It is odd, and exact at 0 and +-1 (xi or w is 0).  Its error is that of the
// Newton steps it replaced: 0.29 ulp root mean square, at most 0.51 at
// dt = 5e-4 and 0.53 at 0.05.  Up to dt = 0.45 a polynomial of the same form
// starts one Newton step.  Measured against Newton steps alone, on the tuned
// launches: 24.6 to 19.9 ms per 100 monitored steps at 512^3 (dt = 5e-4), 2.65
// to 2.08 ms per 1000 at 1024^2 (dt = 1e-3).
//
// Larger dt takes Newton's method alone, from the expansion of the root in h
// on a = |xi|, to first order, theta_0 = a - h f(a) = a + h a (1 - a^2), or
// (c.start2) to second order, theta_0 = a - h f(a) (1 - h f'(a)) with
// f' = 3 a^2 - 1, and `nit` steps; the host picks the start and nit by
// running this same iteration in extended precision over a <= 1.  When
// h > 1/2 the expansion is poor and the start is a itself: the expansion's h
// is then c.hs = 0, which gives a exactly (a + 0 * (finite) = a), so no lane
// selects.  For |xi| > 1 (only when the conditions fail) the iteration starts
// from a, takes the same `nit` steps and continues until the correction stops
// mattering (at most 200 more steps).

// Reciprocal of a positive double near [0.5, 4]: hardware estimate plus one
// Newton-Raphson correction.  Only used for Newton steps on the cubic, whose
// own iteration absorbs the remaining error.
__device__ __forceinline__ double approx_rcp(double d)
{
    double r = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, r, 1.0);
    r = fma(r, e, r);
    return r;
}

template <bool S2>
__device__ __forceinline__ double root_start_t(double a, const StepCoef &c)
{
    if (S2) {
        const double a2 = a * a;
        const double f = fma(a2, a, -a);        // f(a)
        const double t = fma(-c.h3, a2, c.oph);  // 1 - h f'(a)
        return fma(-(c.hs * f), t, a);
    }
    return fma(c.hs * a, fma(-a, a, 1.0), a);
}

__device__ __forceinline__ double root_start(double a, const StepCoef &c)
{
    return c.start2 ? root_start_t<true>(a, c) : root_start_t<false>(a, c);
}

// A copy of c with omh held in vector registers for the variants whose common
// path takes Newton steps: a VOP3 instruction reads at most one scalar
// register, so fma(h3, x^2, omh) with both coefficients in scalar registers
// costs a move at every node; a kernel that passes this copy to the root pays
// it once.  (The empty asm only makes the value look per-lane to the
// compiler; it emits no instruction.)
template <int RV>
__device__ __forceinline__ StepCoef coef_vgpr(const StepCoef &c)
{
    StepCoef v = c;
    if (RV == 0 || (RV <= ROOT_POLYS && ROOT_NEWTON[RV] > 0)) asm volatile("" : "+v"(v.omh));
    return v;
}

// One Newton step on the cubic from x, with the reciprocal of the
// derivative from its hardware estimate and one correction.
__device__ __forceinline__ double newton_step(double x, double a, const StepCoef &c)
{
    const double x2 = x * x;
    const double p = fma(c.h, fma(x, x2, -x), x - a);
    const double dp = fma(c.h3, x2, c.omh);
    return fma(-p, approx_rcp(dp), x);
}

// Newton steps with a true division from x until the correction stops
// mattering (below 2^-54 x; at most 200 steps): the root for a > 1.
__device__ __forceinline__ double newton_converge(double x, double a, const StepCoef &c)
{
    for (int k = 0; k < 200; ++k) {
        const double x2 = x * x;
        const double p = fma(c.h, fma(x, x2, -x), x - a);
        const double dp = fma(c.h3, x2, c.omh);
        const double step = p / dp;
        x -= step;
        if (!(fabs(step) > 0x1p-54 * x)) break;
    }
    return x;
}

// The root's two paths for one xi with the variant fixed at compile time:
// root_common is the root for |xi| <= 1, root_restart the one for |xi| > 1.
// root_restart is the same code in every variant, and the run-time variant
// repeats the compiled one's operations, so every kernel rounds the same.
template <int RV>
__device__ __forceinline__ double root_common(double xi, const StepCoef &c)
{
    if constexpr (RV >= 1 && RV <= ROOT_POLYS) {
        constexpr int D = ROOT_DEG[RV];
        const double w = fma(-xi, xi, 1.0);
        double q = c.q[D];
#pragma unroll
        for (int k = D - 1; k >= 0; --k) q = fma(q, w, c.q[k]);
        double x = fma(xi * w, q, xi);
#pragma unroll
        for (int k = 0; k < ROOT_NEWTON[RV]; ++k) x = newton_step(x, xi, c);
        return x;
    } else {
        const double a = fabs(xi);
        double x = root_start(a, c);
        for (int k = 0; k < c.nit; ++k) x = newton_step(x, a, c);
        return copysign(x, xi);
    }
}

__device__ __forceinline__ double root_restart(double xi, const StepCoef &c)
{
    const double a = fabs(xi);
    double x = a;
#pragma unroll 1
    for (int k = 0; k < c.nit; ++k) x = newton_step(x, a, c);
    return copysign(newton_converge(x, a, c), xi);
}

template <int RV>
__device__ __forceinline__ double cubic_root_n(double xi, const StepCoef &c)
{
    double x = root_common<RV>(xi, c);
    if (fabs(xi) > 1.0) x = root_restart(xi, c);  // this lane's first pass is discarded
    return x;
}

// The root with the variant known only at run time (uniform: one branch).
__device__ __forceinline__ double cubic_root(double xi, const StepCoef &c)
{
    double x = with_root(c.rv, [&](auto RVc) { return root_common<decltype(RVc)::value>(xi, c); });
    if (fabs(xi) > 1.0) x = root_restart(xi, c);
    return x;
}

// The roots of N values with one test for the |xi| > 1 case (on the largest
// |xi|; a NaN never needs it), so the common paths of the N values form one
// block that the compiler can interleave.  Same results as cubic_root_n.
template <int RV, int N>
__device__ __forceinline__ void cubic_roots_n(const double (&xi)[N], double (&th)[N], const StepCoef &c)
{
    if constexpr (RV == ROOT_FEX) {
#pragma unroll
        for (int r = 0; r < N; ++r) th[r] = xi[r];
        return;
    }
    double amax = fabs(xi[0]);
#pragma unroll
    for (int r = 0; r < N; ++r) {
        th[r] = root_common<RV>(xi[r], c);
        if (r > 0) amax = fmax(amax, fabs(xi[r]));
    }
    if (amax > 1.0) {
#pragma unroll
        for (int r = 0; r < N; ++r)
            if (fabs(xi[r]) > 1.0) th[r] = root_restart(xi[r], c);
    }
}

// Explicit part xi from the node value p and the sum over axes of its two
// neighbours' sum (nsum = sum_k (p_{+k} + p_{-k})), for d = D.
template <int D>
__device__ __forceinline__ double explicit_part(double p, double nsum, const StepCoef &c)
{
    const double lap = fma(-2.0 * D, p, nsum);
    const double t = fma(c.kappa, lap, p);
    const double f = fma(p, p * p, -p);
    return fma(-c.h, f, t);
}

// The fully explicit comparison scheme of Sec. 3.3, Remark 2 (FEX-FD):
// phi + kappa sum_k (phi_{+k} + phi_{-k} - 2 phi) - dt f(phi).
template <int D>
__device__ __forceinline__ double explicit_fex(double p, double nsum, const StepCoef &c)
{
    const double lap = fma(-2.0 * D, p, nsum);
    const double t = fma(c.kappa, lap, p);
    const double f = fma(p, p * p, -p);
    return fma(-c.dt, f, t);
}

// The part of the step before the root: xi, or with ROOT_FEX the explicit
// scheme's new value (which needs none).
template <int D, int RV>
__device__ __forceinline__ double explicit_n(double p, double nsum, const StepCoef &c)
{
    return RV == ROOT_FEX ? explicit_fex<D>(p, nsum, c) : explicit_part<D>(p, nsum, c);
}

template <int D>
__device__ __forceinline__ double update(double p, double nsum, const StepCoef &c)
{
    if (c.fex) return explicit_fex<D>(p, nsum, c);
    return cubic_root(explicit_part<D>(p, nsum, c), c);
}

// (a launcher may also give the explicit scheme the run-time variant)
template <int D, int RV>
__device__ __forceinline__ double update_n(double p, double nsum, const StepCoef &c)
{
    if (RV == ROOT_FEX || (RV == 0 && c.fex)) return explicit_fex<D>(p, nsum, c);
    return cubic_root_n<RV>(explicit_part<D>(p, nsum, c), c);
}

// Value used for an out-of-range neighbour (rows of the paper's D matrices):
// Neumann mirrors the node itself, Dirichlet reads the zero wall, periodic
// reads the wrapped node `wrap`.
template <int BC>
__device__ __forceinline__ double outside(double self, double wrap)
{
    if (BC == BC_HN) return self;
    if (BC == BC_HD) return 0.0;
    return wrap;
}

// NaN-propagating maximum (fmax drops NaN).
// Workgroups are dealt to the 8 XCDs round-robin: block b runs on XCD b % 8.
// This renumbering gives each XCD one contiguous range of logical tiles, so
// neighbouring tiles, which read each other's edge rows, share that XCD's L2.
// It is a bijection on [0, nblk) for every nblk: with nblk = 8q + r, XCDs
// 0..r-1 take q+1 tiles and the others q.
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nblk)
{
    const int64_t q = nblk >> 3, r = nblk & 7, x = b & 7, k = b >> 3;
    return (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + k;
}

__device__ __forceinline__ double nan_max(double a, double b)
{
    if (a != a) return a;
    if (b != b) return b;
    return a > b ? a : b;
}

// Monitor terms of one node with value p: bulk (p^2 - 1)^2 / 4; the squared
// difference along each axis to the next node (the BC's value past the last
// node, so HN adds 0, HD adds p^2 for the wall edge, P adds the wrap edge);
// HD also adds p^2 for the wall edge before the first node.
struct MonAcc {
    double bulk, grad, mx;
};

__device__ __forceinline__ void mon_zero(MonAcc &m)
{
    m.bulk = 0.0;
    m.grad = 0.0;
    m.mx = 0.0;
}

__device__ __forceinline__ double bulk_term(double p)
{
    const double q = fma(p, p, -1.0);
    return 0.25 * (q * q);
}

// Wave64 butterfly sums: every lane ends with the same, order-fixed value.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = nan_max(v, __shfl_xor(v, o, 64));
    return v;
}

// Deterministic block reduction of (bulk, grad, max); thread 0 writes the
// triple to out[0..2].  `lds` holds 3 * (blockDim / 64) doubles.
__device__ __forceinline__ void block_reduce_store(MonAcc m, double *lds, double *out)
{
    const int lane = threadIdx.x & 63;
    const int nthreads = blockDim.x * blockDim.y * blockDim.z;
    const int tid = threadIdx.x + blockDim.x * (threadIdx.y + blockDim.y * threadIdx.z);
    const int wave = tid >> 6;
    const int nw = (nthreads + 63) >> 6;
    (void)lane;
    const double b = wave_sum(m.bulk);
    const double g = wave_sum(m.grad);
    const double x = wave_max(m.mx);
    if ((tid & 63) == 0) {
        lds[3 * wave + 0] = b;
        lds[3 * wave + 1] = g;
        lds[3 * wave + 2] = x;
    }
    __syncthreads();
    if (tid == 0) {
        double sb = 0.0, sg = 0.0, sx = 0.0;
        for (int w = 0; w < nw; ++w) {
            sb += lds[3 * w + 0];
            sg += lds[3 * w + 1];
            sx = nan_max(sx, lds[3 * w + 2]);
        }
        out[0] = sb;
        out[1] = sg;
        out[2] = sx;
    }
}

}  // namespace ace
