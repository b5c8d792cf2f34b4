// Reverse sweep of a 2D field on register-resident regions, and the recompute
// of the states it needs next, in one launch.
//
// A launch holds two kinds of workgroups on the same (RH - 2K) x (64 - 2K)
// tiles (ace_tb2.h): the first n_rev take Sr <= K transposed steps of one
// checkpoint segment, the others Sf <= K forward steps of the segment before
// it, writing every level.  The two are independent, so one fills the CUs the
// other leaves idle without a second stream and its events, and a segment
// costs as many host calls as it has launches.
//
// The transposed step works on mu = lambda R'(xi) instead of lambda: with
// jd = 1 - h (3 phi^2 - 1) and r = 1 / (1 + h (3 phi^2 - 1)) of the state phi^n,
//   lambda^n = jd mu^{n+1} + kappa Lambda mu^{n+1},   mu^n = lambda^n r,
// so each state is read once, at its own nodes, and mu is evaluated once per
// node.  mu passes between launches; the first takes lambda^T and phi^T, the
// last writes lambda^0.  Boundary images as in the forward step: mu is even at
// Neumann and odd at Dirichlet walls, phi enters squared.  dL/dkappa sums
// (phi^n - b) Lambda mu (Lambda is symmetric), so phi's neighbours are not
// needed.  Without Dirichlet walls Lambda's columns sum to 0 and any b gives the
// same sum: b is the state's first value if a node in the middle holds it too,
// so that a uniform field's gradient is 0 as that of mu Lambda phi^n is and not
// a residue of Lambda mu's roundings, and 0 otherwise.
//
// Bound: the states' bytes and the region levels' issue, about equally.  512^2
// with 32-step segments: 15.5 us per launch of 8 transposed and 8 recomputed
// steps (the 33 MB of states written and read 7 us at the rate of a copy, the
// recompute alone 11.6), 2.0 ms per 1000 steps; on LDS regions, with the
// recompute on a second stream and 14 host calls per segment, 3.3.
#include <type_traits>

#include "ace_tb2.h"

namespace ace {

namespace {

using tb2::Geom;
using tb2::lane_shift;
using tb2::Region;
using tb2::RX;

// 1 / (1 + h (3 p^2 - 1)): the hardware estimate refined by two Newton-Raphson
// steps, as everywhere in the reverse sweep.
__device__ __forceinline__ double dprime(double p2, const StepCoef &c)
{
    const double dp = fma(c.h3, p2, c.omh);
    double r = __builtin_amdgcn_rcp(dp);
    r = fma(r, fma(-dp, r, 1.0), r);
    return fma(r, fma(-dp, r, 1.0), r);
}

// One lane's value, in scalar registers.
__device__ __forceinline__ double lane_value(double v, int lane)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u & 0xffffffffull), lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int BC, int RV, int TRW, int RYT>
__global__ __launch_bounds__(RX * TRW) void k_adj2(Shape s, StepCoef c0, Adj2Args a, int tiles_x)
{
    constexpr int RH = Geom<TRW, RYT>::RH;
    __shared__ double EB[2 * 2 * TRW * RX];
    __shared__ double red[TRW];
    const StepCoef c = coef_vgpr<RV>(c0);
    const int K = a.K;
    int b = (int)xcd_tile(blockIdx.x, gridDim.x);
    if (b >= a.n_rev) {  // recompute
        b -= a.n_rev;
        const Region<BC, TRW, RYT> g(s, K, b / tiles_x, b - (b / tiles_x) * tiles_x);
        double v[RYT];
        g.load(s, a.f_in, v);
        MonAcc m;
        mon_zero(m);
        g.template advance<false, true, RV>(s, c, v, a.f_out, a.stride, EB, m, a.Sf);
        return;
    }
    const Region<BC, TRW, RYT> g(s, K, b / tiles_x, b - (b / tiles_x) * tiles_x);
    const int tx = g.tx, tr = g.tr, S = a.Sr;
    auto eb = [&](int par, int side, int w) -> double * { return EB + ((par * 2 + side) * TRW + w) * RX; };
    int oof[RYT];
#pragma unroll
    for (int r = 0; r < RYT; ++r) {
        const int ry = tr * RYT + r, yg = g.yr0 + ry;
        oof[r] = (g.xin && ry >= K && ry < RH - K && yg >= 0 && yg < g.M1) ? yg * g.M2 + g.xg : -1;
    }
    // where this thread's nodes of a state lie (its square and, in the domain,
    // its value are used: images need no sign)
    int off[RYT];
#pragma unroll
    for (int r = 0; r < RYT; ++r) {
        int sy;
        off[r] = tb2::image<BC>(g.yr0 + tr * RYT + r, g.M1, sy) * g.M2 + g.mx;
    }
    // level t (1..S) uses phi^{m+S-t}, in slot t % 4, loaded three levels ahead
    // (a level takes under 1 us, a load from another XCD's cache over 1)
    double v[RYT], ph[4][RYT], base[4];
    // (lane 0 holds a state's first value, the others the middle one)
    const int probe = tx == 0 ? 0 : (g.M1 / 2) * g.M2 + g.M2 / 2;
    auto fetch = [&](int t, double(&dst)[RYT], double &b) {
        const double *p = t >= S ? a.phi_first : a.phi_rest + (int64_t)(S - t - 1) * a.stride;
#pragma unroll
        for (int r = 0; r < RYT; ++r) dst[r] = p[off[r]];
        if (BC != BC_HD) b = p[probe];
    };
    g.load(s, a.mu_in, v);
    if (a.phi_end) {
#pragma unroll
        for (int r = 0; r < RYT; ++r) ph[0][r] = a.phi_end[off[r]];
    }
    fetch(1, ph[1], base[1]);
    fetch(2, ph[2], base[2]);
    fetch(3, ph[3], base[3]);
    if (a.phi_end) {  // lambda^T: its mu from phi^T
#pragma unroll
        for (int r = 0; r < RYT; ++r) v[r] *= dprime(ph[0][r] * ph[0][r], c);
    }
    eb(0, 0, tr)[tx] = v[0];
    eb(0, 1, tr)[tx] = v[RYT - 1];
    __syncthreads();
    const int H = g.M1 - g.yr0 + S < RH ? g.M1 - g.yr0 + S : RH;
    double gs = 0.0;
    int t = 1;
    auto level = [&](const double(&p_)[RYT], double b, double(&next)[RYT], double &next_b)
                     __attribute__((always_inline)) -> bool {
        const double b0 = BC != BC_HD && lane_value(b, 0) == lane_value(b, 1) ? lane_value(b, 0) : 0.0;
        if (t + 3 <= S) fetch(t + 3, next, next_b);
        const int rd = (t - 1) & 1;
        const double eT = eb(rd, 1, tr > 0 ? tr - 1 : 0)[tx];
        const double eB = eb(rd, 0, tr < TRW - 1 ? tr + 1 : TRW - 1)[tx];
        // all rows of a wavefront together where all are needed at this level
        // (their chains interleave), else row by row (wave-uniform tests)
        auto rows = [&](auto FULLc) __attribute__((always_inline)) {
            constexpr bool FULL = decltype(FULLc)::value;
            double lam[RYT], rp[RYT];
#pragma unroll
            for (int r = 0; r < RYT; ++r) {
                lam[r] = v[r];
                rp[r] = 1.0;
                const int ry = tr * RYT + r;
                if (!FULL && (ry < t || ry >= H - t)) continue;
                const double mu = v[r], p = p_[r];
                const double ym = (r > 0) ? v[r > 0 ? r - 1 : 0] : eT;
                const double yp = (r < RYT - 1) ? v[r < RYT - 1 ? r + 1 : 0] : eB;
                const double msum = (ym + yp) + (lane_shift<0x138>(mu) + lane_shift<0x130>(mu));
                const double lap = fma(-4.0, mu, msum);
                const double p2 = p * p;
                const double jd = fma(-c.h3, p2, c.oph);
                lam[r] = fma(c.kappa, lap, jd * mu);
                rp[r] = dprime(p2, c);
                gs = fma(oof[r] >= 0 ? p - b0 : 0.0, lap, gs);
            }
            const bool write_lambda = t == S && a.last;
#pragma unroll
            for (int r = 0; r < RYT; ++r) v[r] = write_lambda ? lam[r] : lam[r] * rp[r];
        };
        const int row0 = tr * RYT;
        if (row0 >= t && row0 + RYT <= H - t) rows(std::true_type());
        else rows(std::false_type());
        if (t == S) return true;
        eb(t & 1, 0, tr)[tx] = v[0];
        eb(t & 1, 1, tr)[tx] = v[RYT - 1];
        __syncthreads();
        ++t;
        return false;
    };
    for (;;) {
        if (level(ph[1], base[1], ph[0], base[0])) break;
        if (level(ph[2], base[2], ph[1], base[1])) break;
        if (level(ph[3], base[3], ph[2], base[2])) break;
        if (level(ph[0], base[0], ph[3], base[3])) break;
    }
#pragma unroll
    for (int r = 0; r < RYT; ++r)
        if (oof[r] >= 0) a.mu_out[oof[r]] = v[r];
    gs = wave_sum(gs);
    if (tx == 0) red[tr] = gs;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = red[0];
        for (int w = 1; w < TRW; ++w) t += red[w];
        a.gpart[b] = a.accumulate ? a.gpart[b] + t : t;
    }
}

template <int RYT>
hipError_t launch(const Shape &s, const StepCoef &c, const Adj2Args &a, hipStream_t st)
{
    constexpr int TRW = ADJ2_THREADS / 64;
    int tiles_x, n;
    tb2::tiles<TRW, RYT>(s, a.K, tiles_x, n);
    if (a.n_rev != 0 && a.n_rev != n) return hipErrorInvalidValue;
    const int nblk = a.n_rev + (a.Sf > 0 ? n : 0);
    auto by_rv = [&](auto BCc) {
        return with_root(c.rv, [&](auto RVc) {
            constexpr int RV = decltype(RVc)::value;  // (no reverse sweep of the explicit scheme)
            hipLaunchKernelGGL((k_adj2<decltype(BCc)::value, RV == ROOT_FEX ? 0 : RV, TRW, RYT>), dim3(nblk),
                               dim3(RX * TRW), 0, st, s, c, a, tiles_x);
            return hipGetLastError();
        });
    };
    switch (s.bc) {
    case BC_HN: return by_rv(RootTag<BC_HN>());
    case BC_HD: return by_rv(RootTag<BC_HD>());
    case BC_P: return by_rv(RootTag<BC_P>());
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

int64_t adj2_tiles(const Shape &s, int rows, int K)
{
    int tiles_x, n;
    if (rows == 64) tb2::tiles<16, 4>(s, K, tiles_x, n);
    else tb2::tiles<16, 2>(s, K, tiles_x, n);
    return n;
}

hipError_t launch_adj2(int rows, const Shape &s, const StepCoef &c, const Adj2Args &a, hipStream_t st)
{
    if (!tb2_supported(s) || (rows != 32 && rows != 64) || a.K < 1 || a.K > rows / 2 - 4 || a.Sr < 0 || a.Sr > a.K ||
        a.Sf < 0 || a.Sf > a.K || (a.n_rev > 0) != (a.Sr > 0) || (a.Sr == 0 && a.Sf == 0))
        return hipErrorInvalidValue;
    return rows == 64 ? launch<4>(s, c, a, st) : launch<2>(s, c, a, st);
}

}  // namespace ace
