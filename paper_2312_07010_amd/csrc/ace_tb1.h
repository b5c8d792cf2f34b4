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

}  // namespace tb1
}  // namespace ace
