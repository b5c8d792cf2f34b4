// One 3D step with neighbours through the cache, several planes per thread.
//
// A thread owns one column (i1, i2) of Z consecutive planes: it loads the
// Z + 2 values of its column once and its four in-plane neighbours per plane,
// all before the first update, so the whole input of a wavefront is in
// flight at once.  Columns are numbered flat over the plane (64 consecutive
// i1 M2 + i2 per wavefront): ragged planes leave no lanes idle and every load
// of a wavefront covers at most five cache lines more than the least.  The
// in-plane offsets are 32-bit and found once per thread; an offset past the
// plane makes the buffer load return 0, which is the Dirichlet wall, and a
// Neumann neighbour past the end is the node itself.
//
// Bound: fields up to a few million nodes stay in the caches and a step is
// launch pace (2.2 us) plus one round of load latency.  With one node per
// thread and 64-bit coordinates a step of 64^3 took 3.3 us, 72 x 61 x 80
// (Dirichlet) 6.0, 96^3 9.2 and 130^3 18.1.
#include "ace_col.h"

namespace ace {

namespace {

using namespace col;

template <int BC, bool MON, int RV, int Z>
__global__ __launch_bounds__(CNT) void k_col3d(int M0, int M1, int M2, int nb, StepCoef c,
                                               const double *__restrict__ in, double *__restrict__ out,
                                               double *__restrict__ partials)
{
    __shared__ double red[3 * (CNT / 64)];
    // plane chunks outermost, so an XCD's workgroups share planes
    const int t = (int)xcd_tile(blockIdx.x, gridDim.x);
    const int PS = M1 * M2;
    const int z0 = (t / nb) * Z;
    const int nz = M0 - z0 < Z ? M0 - z0 : Z;
    const Col k = column<BC>((t - (t / nb) * nb) * CNT + (int)threadIdx.x, M1, M2);
    double q[Z + 2], ym[Z], yp[Z], xm[Z], xp[Z];
    q[0] = load(plane_at<BC>(in, z0 - 1, M0, PS), k.o);
#pragma unroll
    for (int i = 0; i < Z; ++i) {
        // (planes past the last one repeat it: loaded, not used)
        const __amdgpu_buffer_rsrc_t r = plane_at<BC>(in, i < nz ? z0 + i : z0 + nz, M0, PS);
        q[i + 1] = load(r, k.o);
        ym[i] = load(r, k.ym);
        yp[i] = load(r, k.yp);
        xm[i] = load(r, k.xm);
        xp[i] = load(r, k.xp);
    }
    q[Z + 1] = load(plane_at<BC>(in, z0 + nz, M0, PS), k.o);
    double xi[Z], th[Z];
#pragma unroll
    for (int i = 0; i < Z; ++i) {
        const double nsum = ((q[i] + q[i + 2]) + (ym[i] + yp[i])) + (xm[i] + xp[i]);
        xi[i] = explicit_n<3, RV>(q[i + 1], nsum, c);
    }
    cubic_roots_n<RV>(xi, th, c);
    MonAcc m;
    mon_zero(m);
#pragma unroll
    for (int i = 0; i < Z; ++i) {
        if (i >= nz) break;
        const __amdgpu_buffer_rsrc_t r = plane_rsrc(out + (int64_t)(z0 + i) * PS, PS * 8);
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(BufB64, th[i]), r, (int)k.o, 0, 0);
        if (MON && k.o != kNone) {
            const double p = q[i + 1], dz = q[i + 2] - p, dy = yp[i] - p, dx = xp[i] - p;
            double g = fma(dz, dz, fma(dy, dy, dx * dx));
            if (BC == BC_HD) {
                if (z0 + i == 0) g = fma(p, p, g);
                if (k.y0) g = fma(p, p, g);
                if (k.x0) g = fma(p, p, g);
            }
            m.bulk += bulk_term(p);
            m.grad += g;
            m.mx = nan_max(m.mx, fabs(p));
        }
    }
    if (MON) block_reduce_store(m, red, partials + 3 * t);
}

// Planes per thread: as many as keep two workgroups on each of 256 CUs
// (more reuse of the column's values), at least 2.
int planes_per_thread(const Shape &s)
{
    const int64_t nb = (s.M1 * s.M2 + CNT - 1) / CNT;
    for (int Z : {8, 4})
        if (nb * ((s.M0 + Z - 1) / Z) >= 512) return Z;
    return 2;
}

int64_t blocks(const Shape &s, int Z)
{
    return ((s.M1 * s.M2 + CNT - 1) / CNT) * ((s.M0 + Z - 1) / Z);
}

}  // namespace

// (in-plane byte offsets are 32-bit; the root of a run-time Newton count is
// in the compiled variants too)
bool col3d_supported(const Shape &s)
{
    return s.d == 3 && s.M1 * s.M2 < ((int64_t)1 << 28) && s.M0 < INT32_MAX &&
           blocks(s, planes_per_thread(s)) <= max_blocks(CNT);
}

int64_t col3d_partials_needed(const Shape &s) { return blocks(s, planes_per_thread(s)); }

hipError_t launch_step_col3d(const Shape &s, const StepCoef &c, const double *in, double *out, double *partials,
                             int64_t *nparts, hipStream_t st)
{
    if (!col3d_supported(s)) return hipErrorInvalidValue;
    const int Z = planes_per_thread(s);
    const int64_t nblk = blocks(s, Z);
    const int nb = (int)((s.M1 * s.M2 + CNT - 1) / CNT);
    if (nparts) *nparts = nblk;
    auto go = [&](auto BCc, auto Zc) {
        return with_root(c.rv, [&](auto RVc) {
            constexpr int B = decltype(BCc)::value, ZZ = decltype(Zc)::value, RV = decltype(RVc)::value;
            if (partials)
                hipLaunchKernelGGL((k_col3d<B, true, RV, ZZ>), dim3((unsigned)nblk), dim3(CNT), 0, st, (int)s.M0,
                                   (int)s.M1, (int)s.M2, nb, c, in, out, partials);
            else
                hipLaunchKernelGGL((k_col3d<B, false, RV, ZZ>), dim3((unsigned)nblk), dim3(CNT), 0, st, (int)s.M0,
                                   (int)s.M1, (int)s.M2, nb, c, in, out, partials);
            return hipGetLastError();
        });
    };
    auto by_z = [&](auto BCc) {
        if (Z == 8) return go(BCc, RootTag<8>());
        if (Z == 4) return go(BCc, RootTag<4>());
        return go(BCc, RootTag<2>());
    };
    switch (s.bc) {
    case BC_HN: return by_z(RootTag<BC_HN>());
    case BC_HD: return by_z(RootTag<BC_HD>());
    case BC_P: return by_z(RootTag<BC_P>());
    default: return hipErrorInvalidValue;
    }
}

}  // namespace ace
