// 1D kernels on register-resident segments (ace_tb1.h): K steps per launch
// with one wavefront per segment (any size), and all steps of a small field
// in one workgroup.
#include <algorithm>

#include "ace_tb1.h"

namespace ace {

namespace {

// K steps (1 <= K < 32 R) from in to out, one wavefront per workgroup; MON:
// the monitor partial of each wavefront's output nodes of `in`.
template <int BC, bool MON, int RV, int R>
__global__ __launch_bounds__(64) void k_tb1(int n, StepCoef c0, const double *__restrict__ in,
                                            double *__restrict__ out, double *__restrict__ partials, int K)
{
    const StepCoef c = coef_vgpr<RV>(c0);
    const int o0 = (int)blockIdx.x * (64 * R - 2 * K);  // first output node
    const int o1 = o0 + 64 * R - 2 * K < n ? o0 + 64 * R - 2 * K : n;
    const int first = o0 - K + (int)threadIdx.x * R;
    double v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int sg;
        const double x = in[tb1::source<BC>(first + r, n, sg)];
        v[r] = (BC != BC_HD || sg > 0) ? x : (sg < 0 ? -x : 0.0);
    }
    auto own = [&](int i) { return i >= o0 && i < o1; };
    if (MON) {
        MonAcc m;
        mon_zero(m);
        tb1::monitor<BC>(v, first, own, m);
        const double b = wave_sum(m.bulk), g = wave_sum(m.grad), x = wave_max(m.mx);
        if (threadIdx.x == 0) {
            partials[3 * blockIdx.x + 0] = b;
            partials[3 * blockIdx.x + 1] = g;
            partials[3 * blockIdx.x + 2] = x;
        }
    }
    for (int k = 0; k < K; ++k) tb1::step<R, RV>(v, c);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (own(first + r)) out[first + r] = v[r];
}

// All steps of a field of up to R1_MAX nodes in one workgroup: each
// wavefront advances its segment `K` steps in registers, then the wavefronts
// exchange their output nodes through LDS (two buffers, one barrier).  A
// step of the one-node-per-thread kernel (k_resident) waits for the barrier,
// LDS and the dependent chain of a node each time, 0.35 us at 256 nodes; here
// the chain is left.
template <int BC, int RV, int R>
__global__ __launch_bounds__(64 * R1_WAVES) void k_resident1(int n, StepCoef c0, double *__restrict__ field,
                                                            int64_t nsteps, int64_t every, double *__restrict__ mon,
                                                            int K)
{
    __shared__ double fb[2 * (R1_MAX + 1)];
    __shared__ double red[3 * R1_WAVES];
    const StepCoef c = coef_vgpr<RV>(c0);
    if (every > 0) tb1::resident<BC, RV, R, true>(n, c, field, nsteps, every, mon, K, fb, R1_MAX + 1, red);
    else tb1::resident<BC, RV, R, false>(n, c, field, nsteps, 0, nullptr, K, fb, R1_MAX + 1, red);
}

template <class F>
auto with_bc_r(int bc, int R, F &&f)
{
    auto by_r = [&](auto B) {
        switch (R) {
        case 1: return f(B, RootTag<1>());
        case 2: return f(B, RootTag<2>());
        default: return f(B, RootTag<4>());
        }
    };
    switch (bc) {
    case BC_HN: return by_r(RootTag<BC_HN>());
    case BC_HD: return by_r(RootTag<BC_HD>());
    default: return by_r(RootTag<BC_P>());
    }
}

}  // namespace

bool tb1_supported(const Shape &s) { return s.d == 1 && s.M2 < ((int64_t)1 << 30) - 1; }

int64_t tb1_blocks(const Shape &s, int R, int K) { return (s.M2 + 64 * R - 2 * K - 1) / (64 * R - 2 * K); }

hipError_t launch_step_tb1(const Shape &s, const StepCoef &c, const double *in, double *out, double *partials,
                           int64_t *nparts, int R, int K, hipStream_t st)
{
    if (!tb1_supported(s) || (R != 1 && R != 2 && R != 4) || K < 1 || K >= 32 * R) return hipErrorInvalidValue;
    const int64_t nblk = tb1_blocks(s, R, K);
    if (nparts) *nparts = nblk;
    return with_bc_r(s.bc, R, [&](auto BCc, auto Rc) {
        return with_root(c.rv, [&](auto RVc) {
            constexpr int B = decltype(BCc)::value, RR = decltype(Rc)::value, RV = decltype(RVc)::value;
            if (partials)
                hipLaunchKernelGGL((k_tb1<B, true, RV, RR>), dim3((unsigned)nblk), dim3(64), 0, st, (int)s.M2, c, in,
                                   out, partials, K);
            else
                hipLaunchKernelGGL((k_tb1<B, false, RV, RR>), dim3((unsigned)nblk), dim3(64), 0, st, (int)s.M2, c, in,
                                   out, partials, K);
            return hipGetLastError();
        });
    });
}

hipError_t launch_resident1(const Shape &s, const StepCoef &c, double *field, int64_t nsteps, int64_t every,
                            double *mon, int R, int K, hipStream_t st)
{
    if (!tb1_supported(s) || s.M2 > R1_MAX || (R != 1 && R != 2 && R != 4) || K < 1 || K >= 32 * R)
        return hipErrorInvalidValue;
    const int64_t waves = tb1_blocks(s, R, K);
    if (waves > R1_WAVES) return hipErrorInvalidValue;
    return with_bc_r(s.bc, R, [&](auto BCc, auto Rc) {
        return with_root(c.rv, [&](auto RVc) {
            constexpr int B = decltype(BCc)::value, RR = decltype(Rc)::value, RV = decltype(RVc)::value;
            hipLaunchKernelGGL((k_resident1<B, RV, RR>), dim3(1), dim3((unsigned)(64 * waves)), 0, st, (int)s.M2, c,
                               field, nsteps, every, mon, K);
            return hipGetLastError();
        });
    });
}

}  // namespace ace
