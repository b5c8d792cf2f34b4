// 1D temporal blocking in registers: one wavefront advances a segment of
// 64 R nodes K steps without LDS or barriers.
//
// Lane x holds the R consecutive nodes s + x R .. s + x R + R - 1 of a segment
// that starts K nodes before the wavefront's 64 R - 2 K output nodes.  Per
// step a lane needs one value from each neighbouring lane (DPP shifts of its
// first and last node); the two lanes at the segment's ends receive 0, so the
// wrong values move inward one node per step and reach the output's edge only
// after K steps.  Nodes outside the domain are the boundary images of
// ace_tb2.h (periodic wrap, Neumann mirror, negated Dirichlet mirror), which
// the step maps to the images of the stepped field, so no node tests for a
// wall.  The arithmetic is that of the one-step kernel, bit for bit.
#pragma once

#include "ace_device.h"
#include "ace_tb2.h"

namespace ace {
namespace tb1 {

// The stored node a lane's slot r holds: index, and sign (0: a Dirichlet wall
// node).
template <int BC>
__device__ __forceinline__ int source(int c, int n, int &sign)
{
    return tb2::image<BC>(c, n, sign);
}

// One step of the segment.
template <int R, int RV>
__device__ __forceinline__ void step(double (&v)[R], const StepCoef &c)
{
    const double lo = tb2::lane_shift<0x138>(v[R - 1]);
    const double hi = tb2::lane_shift<0x130>(v[0]);
    double xi[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double nsum = (r > 0 ? v[r > 0 ? r - 1 : 0] : lo) + (r < R - 1 ? v[r < R - 1 ? r + 1 : 0] : hi);
        xi[r] = explicit_n<1, RV>(v[r], nsum, c);
    }
    cubic_roots_n<RV>(xi, v, c);
}

// Monitor terms of the segment's output nodes (global nodes first ..
// first + R - 1 of this lane; own(i): node i is an output node).
template <int BC, int R, class Own>
__device__ __forceinline__ void monitor(const double (&v)[R], int first, Own own, MonAcc &m)
{
    const double hi = tb2::lane_shift<0x130>(v[0]);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!own(first + r)) continue;
        const double p = v[r], dh = (r < R - 1 ? v[r < R - 1 ? r + 1 : 0] : hi) - p;
        double g = dh * dh;
        if (BC == BC_HD && first + r == 0) g = fma(p, p, g);
        m.bulk += bulk_term(p);
        m.grad += g;
        m.mx = nan_max(m.mx, fabs(p));
    }
}

// All `nsteps` steps of a field of n nodes in one workgroup of
// ceil(n / (64 R - 2 K)) wavefronts (at most; further ones only keep the
// barriers), in place: each wavefront advances its segment up to K steps in
// registers, then the wavefronts exchange their output nodes through the two
// LDS buffers fb[0 .. stride) and fb[stride .. 2 stride), stride > n.  MON:
// the monitor triple of steps 0, every, ... to mon[3 j ...] (red: LDS of
// block_reduce_store).
template <int BC, int RV, int R, bool MON>
__device__ __forceinline__ void resident(int n, const StepCoef &c, double *__restrict__ field, int64_t nsteps,
                                         int64_t every, double *__restrict__ mon, int K, double *fb, int stride,
                                         double *red)
{
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int o0 = wave * (64 * R - 2 * K);
    const int o1 = o0 + 64 * R - 2 * K < n ? o0 + 64 * R - 2 * K : n;
    const int first = o0 - K + lane * R;
    // where this lane's nodes come from: slot n of the buffers holds 0, the
    // Dirichlet wall
    int src[R], sgn[R];
    double v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        src[r] = source<BC>(first + r, n, sgn[r]);
        const double x = field[src[r]];
        v[r] = (BC != BC_HD || sgn[r] > 0) ? x : (sgn[r] < 0 ? -x : 0.0);
        if (BC == BC_HD && sgn[r] == 0) src[r] = n;
    }
    if (threadIdx.x == 0) {
        fb[n] = 0.0;
        fb[stride + n] = 0.0;
    }
    auto own = [&](int i) { return i >= o0 && i < o1; };
    int64_t jm = 0, done = 0;
    int64_t due = MON ? 0 : nsteps + 1;  // next monitored step
    double *f = fb, *g = fb + stride;
    for (;;) {
        if (MON && done == due) {
            MonAcc m;
            mon_zero(m);
            monitor<BC>(v, first, own, m);
            __syncthreads();  // every thread is past the last use of red
            block_reduce_store(m, red, mon + 3 * jm);
            ++jm;
            due += every;
        }
        if (done >= nsteps) break;
        // up to the next monitor in rounds of equal length
        const int64_t left = (due < nsteps ? due : nsteps) - done;
        const int rounds = (int)((left + K - 1) / K);
        const int kb = (int)((left + rounds - 1) / rounds);
        for (int k = 0; k < kb; ++k) step<R, RV>(v, c);
        done += kb;
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (own(first + r)) f[first + r] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double x = f[src[r]];
            v[r] = (BC == BC_HD && sgn[r] < 0) ? -x : x;
        }
        double *const t = f;
        f = g;
        g = t;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (own(first + r)) field[first + r] = v[r];
}

}  // namespace tb1
}  // namespace ace
