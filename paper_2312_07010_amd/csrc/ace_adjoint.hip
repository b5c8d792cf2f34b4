// Transposed step of the scheme (reverse sweep of the time loop).
//
// Forward: phi^{n+1}_i = R(xi_i), xi = phi + kappa Lambda phi - h f(phi), with R
// the root of theta + h (theta^3 - theta) = xi.  Implicit differentiation of
// the cubic gives R'(xi) = 1 / (1 + h (3 theta^2 - 1)).  The Jacobian of xi is
// diag(1 - h (3 phi^2 - 1)) + kappa Lambda and Lambda is symmetric (the D
// matrices of Sec. 2 are), so with mu = lambda^{n+1} R'(xi):
//   lambda^n = (1 - h (3 (phi^n)^2 - 1)) mu + kappa Lambda mu,
//   dL/dkappa += < mu, Lambda phi^n >.
// mu at the neighbours is recomputed from lambda^{n+1} and phi^{n+1} instead
// of being stored, so one pass reads three fields and writes one.
#include "ace_col.h"

namespace ace {

namespace {

constexpr int kBlock = 256;

// mu = lambda R'(xi) = lambda / (1 + h (3 p1^2 - 1)), p1 = phi^{n+1}.  The
// denominator lies in [1 - h, 1 + 2h]; its reciprocal is the hardware estimate
// refined by two Newton-Raphson steps (quadratic convergence takes the
// estimate's error below double rounding).
__device__ __forceinline__ double mu_of(double lam, double p1, const StepCoef &c)
{
    const double dp = fma(c.h3, p1 * p1, c.omh);
    double r = __builtin_amdgcn_rcp(dp);
    r = fma(r, fma(-dp, r, 1.0), r);
    r = fma(r, fma(-dp, r, 1.0), r);
    return lam * r;
}

template <int D, int BC>
__global__ __launch_bounds__(kBlock) void k_adjoint(Shape s, StepCoef c,
                                                    const double *__restrict__ lam,
                                                    const double *__restrict__ phin,
                                                    const double *__restrict__ phin1,
                                                    double *__restrict__ lam_out,
                                                    double *__restrict__ gpart)
{
    __shared__ double lds[kBlock / 64];
    const int64_t i2 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i1 = (int64_t)blockIdx.y * blockDim.y + threadIdx.y;
    const int64_t i0 = blockIdx.z;
    double g = 0.0;
    if (i2 < s.M2 && i1 < s.M1) {
        const int64_t idx = (i0 * s.M1 + i1) * s.M2 + i2;
        const double mu = mu_of(lam[idx], phin1[idx], c);
        const double p = phin[idx];
        const int64_t coord[3] = {i0, i1, i2};
        const int64_t size[3] = {s.M0, s.M1, s.M2};
        const int64_t stride[3] = {s.M1 * s.M2, s.M2, 1};
        double msum = 0.0, psum = 0.0;
#pragma unroll
        for (int a = 3 - D; a < 3; ++a) {
            const int64_t cc = coord[a], n = size[a], st = stride[a];
            double mlo, mhi, plo, phi;
            if (cc > 0) {
                mlo = mu_of(lam[idx - st], phin1[idx - st], c);
                plo = phin[idx - st];
            } else if (BC == BC_HN) {
                mlo = mu;
                plo = p;
            } else if (BC == BC_HD) {
                mlo = 0.0;
                plo = 0.0;
            } else {
                const int64_t w = idx + (n - 1) * st;
                mlo = mu_of(lam[w], phin1[w], c);
                plo = phin[w];
            }
            if (cc < n - 1) {
                mhi = mu_of(lam[idx + st], phin1[idx + st], c);
                phi = phin[idx + st];
            } else if (BC == BC_HN) {
                mhi = mu;
                phi = p;
            } else if (BC == BC_HD) {
                mhi = 0.0;
                phi = 0.0;
            } else {
                const int64_t w = idx - (n - 1) * st;
                mhi = mu_of(lam[w], phin1[w], c);
                phi = phin[w];
            }
            msum += mlo + mhi;
            psum += plo + phi;
        }
        const double lap_mu = fma(-2.0 * D, mu, msum);
        const double lap_p = fma(-2.0 * D, p, psum);
        // 1 - h (3 p^2 - 1) = (1 + h) - 3 h p^2
        const double jd = fma(-c.h3, p * p, 1.0 + c.h);
        lam_out[idx] = fma(c.kappa, lap_mu, jd * mu);
        g = mu * lap_p;
    }
    g = wave_sum(g);
    const int tid = threadIdx.x + blockDim.x * threadIdx.y;
    if ((tid & 63) == 0) lds[tid >> 6] = g;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) t += lds[w];
        gpart[blockIdx.x + (int64_t)gridDim.x * (blockIdx.y + (int64_t)gridDim.y * blockIdx.z)] = t;
    }
}

// 3D: the transposed step on mu (ace_adj2.hip), a thread per column of Z planes
// with all its values in flight at once: mu of the node and its neighbours,
// phi of the node.  phi_end: mu_in is lambda, and its mu is taken at every
// node read.  dL/dkappa sums (phi - b) Lambda mu as in 2D.  (k_adjoint reads three fields at seven nodes each and evaluates
// mu at all seven: 16.6 us per step of 96^3, this one 7.9.)
template <int BC, int Z, bool FIRST>
__global__ __launch_bounds__(col::CNT) void k_adjoint_col(int M0, int M1, int M2, int nb, StepCoef c,
                                                          const double *__restrict__ mu_in,
                                                          const double *__restrict__ phi,
                                                          const double *__restrict__ phi_end,
                                                          double *__restrict__ mu_out, double *__restrict__ gpart,
                                                          int last, int accumulate)
{
    __shared__ double lds[col::CNT / 64];
    const int t = (int)xcd_tile(blockIdx.x, gridDim.x);
    const int PS = M1 * M2;
    const int z0 = (t / nb) * Z;
    const int nz = M0 - z0 < Z ? M0 - z0 : Z;
    const col::Col k = col::column<BC>((t - (t / nb) * nb) * col::CNT + (int)threadIdx.x, M1, M2);
    auto at = [&](int z, uint32_t off) -> double {
        const double v = col::load(col::plane_at<BC>(mu_in, z, M0, PS), off);
        if (!FIRST) return v;
        return mu_of(v, col::load(col::plane_at<BC>(phi_end, z, M0, PS), off), c);
    };
    double q[Z + 2], p[Z], ym[Z], yp[Z], xm[Z], xp[Z];
    q[0] = at(z0 - 1, k.o);
#pragma unroll
    for (int i = 0; i < Z; ++i) {
        const int z = i < nz ? z0 + i : z0 + nz;  // (past the last plane: loaded, not used)
        q[i + 1] = at(z, k.o);
        ym[i] = at(z, k.ym);
        yp[i] = at(z, k.yp);
        xm[i] = at(z, k.xm);
        xp[i] = at(z, k.xp);
        p[i] = col::load(col::plane_at<BC>(phi, z, M0, PS), k.o);
    }
    q[Z + 1] = at(z0 + nz, k.o);
    const double mid = phi[(int64_t)(M0 / 2) * PS + (M1 / 2) * M2 + M2 / 2];
    const double b = BC != BC_HD && phi[0] == mid ? mid : 0.0;
    double g = 0.0;
#pragma unroll
    for (int i = 0; i < Z; ++i) {
        if (i >= nz) break;
        const double mu = q[i + 1];
        const double msum = ((q[i] + q[i + 2]) + (ym[i] + yp[i])) + (xm[i] + xp[i]);
        const double lap = fma(-6.0, mu, msum);
        const double jd = fma(-c.h3, p[i] * p[i], 1.0 + c.h);
        double v = fma(c.kappa, lap, jd * mu);
        if (!last) v = mu_of(v, p[i], c);
        const __amdgpu_buffer_rsrc_t r = col::plane_rsrc(mu_out + (int64_t)(z0 + i) * PS, PS * 8);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(col::BufB64, v), r, (int)k.o, 0, 0);
        if (k.o != col::kNone) g = fma(p[i] - b, lap, g);
    }
    g = wave_sum(g);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = g;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double s4 = (lds[0] + lds[1]) + (lds[2] + lds[3]);
        gpart[t] = accumulate ? gpart[t] + s4 : s4;
    }
}

// Planes per thread: 4 where that leaves two workgroups for each of 256 CUs.
int adj_planes(const Shape &s)
{
    return ((s.M1 * s.M2 + col::CNT - 1) / col::CNT) * ((s.M0 + 3) / 4) >= 512 ? 4 : 2;
}

void adj_grid(const Shape &s, dim3 &grid, dim3 &block)
{
    int bx = 1;
    while (bx < s.M2 && bx < kBlock) bx <<= 1;
    if (s.d == 1) bx = kBlock;
    const int by = kBlock / bx;
    block = dim3(bx, by, 1);
    grid = dim3((unsigned)((s.M2 + bx - 1) / bx), (unsigned)((s.M1 + by - 1) / by), (unsigned)s.M0);
}

}  // namespace

int64_t adjoint_partials_needed(const Shape &s)
{
    dim3 grid, block;
    adj_grid(s, grid, block);
    return (int64_t)grid.x * grid.y * grid.z;
}

int64_t adjoint_col_blocks(const Shape &s)
{
    const int Z = adj_planes(s);
    return ((s.M1 * s.M2 + col::CNT - 1) / col::CNT) * ((s.M0 + Z - 1) / Z);
}

bool adjoint_col_supported(const Shape &s)
{
    return col3d_supported(s) && adjoint_col_blocks(s) <= max_blocks(col::CNT);
}

hipError_t launch_adjoint_col(const Shape &s, const StepCoef &c, const double *mu_in, const double *phi,
                              const double *phi_end, double *mu_out, double *gpart, int last, int accumulate,
                              hipStream_t st)
{
    if (!adjoint_col_supported(s)) return hipErrorInvalidValue;
    const int nb = (int)((s.M1 * s.M2 + col::CNT - 1) / col::CNT);
    const dim3 grid((unsigned)adjoint_col_blocks(s));
    auto go = [&](auto BCc, auto Zc) {
        constexpr int B = decltype(BCc)::value, Z = decltype(Zc)::value;
        if (phi_end)
            hipLaunchKernelGGL((k_adjoint_col<B, Z, true>), grid, dim3(col::CNT), 0, st, (int)s.M0, (int)s.M1,
                               (int)s.M2, nb, c, mu_in, phi, phi_end, mu_out, gpart, last, accumulate);
        else
            hipLaunchKernelGGL((k_adjoint_col<B, Z, false>), grid, dim3(col::CNT), 0, st, (int)s.M0, (int)s.M1,
                               (int)s.M2, nb, c, mu_in, phi, phi_end, mu_out, gpart, last, accumulate);
        return hipGetLastError();
    };
    auto by_z = [&](auto BCc) { return adj_planes(s) == 4 ? go(BCc, RootTag<4>()) : go(BCc, RootTag<2>()); };
    switch (s.bc) {
    case BC_HN: return by_z(RootTag<BC_HN>());
    case BC_HD: return by_z(RootTag<BC_HD>());
    case BC_P: return by_z(RootTag<BC_P>());
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_adjoint_step(const Shape &s, const StepCoef &c, const double *lam,
                               const double *phin, const double *phin1, double *lam_out,
                               double *gpart, int64_t *nparts, hipStream_t st)
{
    dim3 grid, block;
    adj_grid(s, grid, block);
    if (nparts) *nparts = (int64_t)grid.x * grid.y * grid.z;
#define ACE_ADJ(DD, BB)                                                                        \
    if (s.d == DD && s.bc == BB) {                                                             \
        hipLaunchKernelGGL((k_adjoint<DD, BB>), grid, block, 0, st, s, c, lam, phin, phin1,    \
                           lam_out, gpart);                                                    \
        return hipGetLastError();                                                              \
    }
    ACE_ADJ(1, BC_HN) ACE_ADJ(1, BC_HD) ACE_ADJ(1, BC_P)
    ACE_ADJ(2, BC_HN) ACE_ADJ(2, BC_HD) ACE_ADJ(2, BC_P)
    ACE_ADJ(3, BC_HN) ACE_ADJ(3, BC_HD) ACE_ADJ(3, BC_P)
#undef ACE_ADJ
    return hipErrorInvalidValue;
}

}  // namespace ace
