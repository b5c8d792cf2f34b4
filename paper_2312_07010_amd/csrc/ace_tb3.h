// 3D step kernel with temporal blocking of depth K (K time levels per HBM
// round trip) on configurable regions.
//
// A workgroup of TRW wavefronts owns an (RH - 2K) x (64 - 2K) output tile of
// the two fastest axes (i1, i2), RH = TRW * RYT, and a chunk of planes along
// i0.  It works on the RH x 64 region around the tile (a ring of K nodes,
// recomputed instead of exchanged) and marches along i0.  Lane x of
// wavefront w holds the RYT consecutive region rows w RYT .. w RYT + RYT - 1
// of column x in registers, for every time level, in register queues along
// i0 (level 0: planes zc-1 .. zc+1, the slot of zc-1 reloaded with plane
// zc+2 as soon as level 1 has read it, about two thirds of a position ahead
// of its use; level j = 1..K-1: the three planes that level j+1 needs
// next).  All queues have three slots, so three march positions fix every
// slot at compile time.  At march position zc it computes level j of plane
// zc - j + 1 for j = 1..K; level K is the output.  Of the seven neighbours of
// a node:
//   * i0: from the level's register queue;
//   * i1 within the thread's rows: registers; across wavefronts (the top and
//     bottom rows of each wavefront's block): LDS edge buffers, one pair per
//     level and march parity (published at position zc, read at zc + 1,
//     with one workgroup barrier per position);
//   * i2: the neighbouring lanes' registers, moved by DPP lane shifts (no LDS
//     round trip on the critical path; the lane at the region edge receives
//     0, a ring node).
// The LDS holds per level only two rows per wavefront.  Every value that
// reaches the output is computed with exactly the arithmetic and neighbour
// order of the one-step kernels, so K steps of this kernel equal K one-step
// launches bit for bit.
//
// Boundary conditions.  Nodes outside the domain are loaded as the images the
// boundary condition makes of the field: periodic wraps; Neumann reflects
// about the wall half a cell past the last node; Dirichlet holds 0 at the wall
// node and the negated reflection beyond it.  The step maps these images to
// the images of the stepped field exactly (the update is odd in (node,
// neighbour sum) and the pair sums are commutative), so at every level every
// node, in the domain or not, takes its plain neighbours with no test per
// node.  With the outward neighbours selected per node at levels >= 2 instead
// (six selects of 64 bits) a Neumann step of 320 x 300 x 310 took 62.9 us.
#pragma once

#include "ace_device.h"

namespace ace {
namespace tb3 {

constexpr int RX = 64;  // region width: one wavefront

// Stored index of the node whose value (times *sign: +1, -1, or 0 for a
// Dirichlet wall node) the boundary condition places at coordinate c of an
// axis of n stored nodes (the ring may reach past the domain more than once
// on tiny grids).  u is c reduced to the images' period (image_period).
template <int BC>
__device__ __forceinline__ int image_period(int n)
{
    return BC == BC_P ? n : (BC == BC_HN ? 2 * n : 2 * (n + 1));
}

template <int BC>
__device__ __forceinline__ int image_of(int u, int n, int &sign)
{
    sign = 1;
    if (BC == BC_P) return u;
    if (BC == BC_HN) return u < n ? u : 2 * n - 1 - u;  // mirror about -1/2 and n - 1/2
    // Dirichlet, u = c + 1 reduced: wall nodes at u = 0 and n + 1
    if (u == 0 || u == n + 1) {
        sign = 0;
        return 0;
    }
    if (u <= n) return u - 1;
    sign = -1;
    return 2 * (n + 1) - u - 1;
}

template <int BC>
__device__ __forceinline__ int image_reduced(int c, int n)
{
    const int P = image_period<BC>(n);
    int u = (BC == BC_HD ? c + 1 : c);
    if (u < 0 || u >= P) {
        u %= P;
        if (u < 0) u += P;
    }
    return u;
}

template <int BC>
__device__ __forceinline__ int image(int c, int n, int &sign)
{
    return image_of<BC>(image_reduced<BC>(c, n), n, sign);
}

// Raw buffer resources over one plane: the fourth descriptor word of
// the gfx9 family, and a byte offset past any plane (2^31, with planes
// below 2^31 bytes), at which a store falls outside the buffer and is
// dropped by the hardware's range check instead of an execution mask.
constexpr int kBufWord3 = 0x00020000;
constexpr uint32_t kNoStore = 0x80000000u;
using BufB64 = decltype(__builtin_amdgcn_raw_buffer_load_b64(__amdgpu_buffer_rsrc_t(), 0, 0, 0));

// The image of a plane index that advances one plane at a time: the stored
// plane's element offset, and its sign, from the reduced index kept up to
// date by a comparison instead of a division per plane.
template <int BC>
struct PlaneCursor {
    int u, sign;
    int64_t off;
    __device__ __forceinline__ void set(int n, int64_t PS) { off = image_of<BC>(u, n, sign) * PS; }
    __device__ __forceinline__ void init(int z0, int n, int64_t PS)
    {
        u = image_reduced<BC>(z0, n);
        set(n, PS);
    }
    __device__ __forceinline__ void next(int n, int64_t PS)
    {
        if (++u == image_period<BC>(n)) u = 0;
        set(n, PS);
    }
};

// The value of the next lower lane (CTRL = 0x138, DPP wave_shr:1) or the next
// higher lane (CTRL = 0x130, wave_shl:1) of a 64-lane wavefront, moved
// between registers by the DPP lane network in two 32-bit halves; lane 0
// (resp. 63) receives 0.
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u & 0xffffffffull), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

template <int K, int TRW, int RYT>
struct Geom {
    static constexpr int NT = RX * TRW;      // threads
    static constexpr int RH = TRW * RYT;     // region rows
    static constexpr int OX = RX - 2 * K;    // output tile width
    static constexpr int OY = RH - 2 * K;    // output tile height
    static constexpr int NQ = K > 1 ? K - 1 : 1;  // level queues 1..K-1
    static_assert(OY >= 4, "region too short for the depth");
};

template <int BC, bool MON, int RV, int K, int TRW, int RYT, int OCC>
__global__ __launch_bounds__(RX * TRW) __attribute__((amdgpu_waves_per_eu(OCC))) void k_tb3(
    Shape s, StepCoef c0, const double *__restrict__ in, double *__restrict__ out,
    double *__restrict__ partials, int tiles_x, int tiles_y, int zchunk)
{
    using G = Geom<K, TRW, RYT>;
    const StepCoef c = coef_vgpr<RV>(c0);
    constexpr int NT = G::NT, RH = G::RH, OX = G::OX, OY = G::OY;
    __shared__ double EB[K * 2 * 2 * TRW * RX];  // [level][parity][top|bottom][wavefront][lane]
    __shared__ double red[3 * (NT / 64)];

    const int tx = threadIdx.x & (RX - 1);
    const int tr = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wavefront index (uniform)
    auto eb = [&](int lvl, int par, int side, int w) -> double * {
        return EB + (((lvl * 2 + par) * 2 + side) * TRW + w) * RX;
    };

    const int64_t t = xcd_tile(blockIdx.x, gridDim.x);  // XCD-aware numbering
    const int64_t ntile = (int64_t)tiles_x * tiles_y;
    int64_t lo, hi;
    if (zchunk > 0) {
        const int64_t tile = t % ntile, chunk = t / ntile;
        lo = tile * s.M0 + chunk * zchunk;
        hi = tile * s.M0 + ((chunk + 1) * zchunk < s.M0 ? (chunk + 1) * zchunk : s.M0);
    } else {
        const int64_t P = ntile * s.M0;
        lo = t * P / gridDim.x;
        hi = (t + 1) * P / gridDim.x;
    }
    const int64_t PS = s.M1 * s.M2;
    MonAcc m;
    mon_zero(m);

    while (lo < hi) {
        const int64_t tile_xy = lo / s.M0;
        const int64_t z0 = lo - tile_xy * s.M0;
        const int64_t z1 = (z0 + (hi - lo) < s.M0) ? z0 + (hi - lo) : s.M0;
        lo += z1 - z0;
        const int tile_x = (int)(tile_xy % tiles_x);
        const int tile_y = (int)(tile_xy / tiles_x);
        const int64_t yr0 = (int64_t)tile_y * OY - K;  // global row of region row 0
        const int64_t xg = (int64_t)tile_x * OX - K + tx;
        int sx;
        const int mxc = image<BC>((int)xg, (int)s.M2, sx);
        const bool xb0 = (xg == 0);

        // per row: in-plane load offset in bytes (kNoStore, past the plane,
        // at a Dirichlet wall: loads 0), its sign bit (Dirichlet images), output
        // offset in bytes (kNoStore: ring or outside the domain), domain-edge
        // flag (uniform)
        uint32_t off[RYT], oof[RYT];
        uint32_t flip[RYT];
        bool yb0[RYT];
#pragma unroll
        for (int r = 0; r < RYT; ++r) {
            const int ry = tr * RYT + r;
            const int64_t yg = yr0 + ry;
            int sy;
            const int myc = image<BC>((int)yg, (int)s.M1, sy);
            off[r] = (BC == BC_HD && sx * sy == 0) ? kNoStore : (uint32_t)(myc * (int)s.M2 + mxc) * 8u;
            flip[r] = sx * sy < 0 ? 0x80000000u : 0u;
            const bool interior = ry >= K && ry < RH - K && tx >= K && tx < RX - K;
            const bool indomain = yg >= 0 && yg < s.M1 && xg >= 0 && xg < s.M2;
            oof[r] = (interior && indomain) ? (uint32_t)(yg * s.M2 + xg) * 8u : kNoStore;
            yb0[r] = (yg == 0);
        }
        // (a buffer over the input plane, empty for a Dirichlet wall plane,
        // and a 32-bit byte offset per lane)
        auto ld = [&](const PlaneCursor<BC> &p, int r) -> double {
            const int bytes = (BC == BC_HD && p.sign == 0) ? 0 : (int)(PS * 8);
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<double *>(in) + p.off, (short)0, bytes, kBufWord3);
            const unsigned long long v = __builtin_bit_cast(
                unsigned long long, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off[r], 0, 0));
            if (BC != BC_HD) return __longlong_as_double((long long)v);
            const uint32_t neg = flip[r] ^ (p.sign < 0 ? 0x80000000u : 0u);
            return __longlong_as_double((long long)(v ^ ((unsigned long long)neg << 32)));
        };

        // level-0 queue: slot k holds plane zs - 1 + k at the first position
        const int64_t zs = z0 - K + 1;           // first march position
        const int64_t zend = z1 + K - 2;         // last march position
        const int64_t zlast = z1 + K - 1;        // last level-0 plane needed
        double q0[3][RYT];
        double qj[G::NQ][3][RYT];
        {
            PlaneCursor<BC> p0, p1, p2;
            p0.init((int)(zs - 1), (int)s.M0, PS);
            p1.init((int)zs, (int)s.M0, PS);
            p2.init((int)(zs + 1), (int)s.M0, PS);
#pragma unroll
            for (int r = 0; r < RYT; ++r) {
                q0[0][r] = ld(p0, r);
                q0[1][r] = ld(p1, r);
                q0[2][r] = ld(p2, r);
            }
        }
#pragma unroll
        for (int j = 0; j < G::NQ; ++j)
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int r = 0; r < RYT; ++r) qj[j][k][r] = 0.0;
        // the plane the next position loads, and the output offset of plane
        // zc - K + 1 (level K's plane)
        static_assert(K >= 2, "the cursor starts at the last plane loaded above");
        PlaneCursor<BC> cur;
        cur.init((int)(zs + 1), (int)s.M0, PS);
        int64_t ooff = (zs - K + 1) * PS;
        // edges of level-0 plane zs, read at the first position
        eb(0, (int)((zs - 1) & 1), 0, tr)[tx] = q0[1][0];
        eb(0, (int)((zs - 1) & 1), 1, tr)[tx] = q0[1][RYT - 1];
        __syncthreads();

        int64_t zc = zs;

        // Level J (1..K) of plane zo = zc - J + 1 from level J-1: zm, cq, zp
        // are the level J-1 values of planes zo-1, zo, zo+1; the result goes
        // to dst (J < K) or to the output (J == K).
        auto level = [&](auto JJ, const double(&zmq)[RYT], const double(&cq)[RYT],
                         const double(&zpq)[RYT], double(&dst)[RYT]) __attribute__((always_inline)) {
            constexpr int J = decltype(JJ)::value;
            const int64_t zo = zc - J + 1;
            const int rd = (int)((zc - 1) & 1);
            // i2 neighbours: the neighbouring lanes' values of the same row
            double xm[RYT], xp[RYT];
#pragma unroll
            for (int r = 0; r < RYT; ++r) {
                xm[r] = lane_shift<0x138>(cq[r]);
                xp[r] = lane_shift<0x130>(cq[r]);
            }
            // i1 neighbours across wavefronts.  Wavefront 0's eT and wavefront
            // TRW-1's eB would lie outside the region: they read their own
            // edge rows instead (in bounds, no branch).  The rows they feed,
            // region rows 0 and RH-1, are ring rows at every level.
            const double eT = eb(J - 1, rd, 1, tr > 0 ? tr - 1 : 0)[tx];
            const double eB = eb(J - 1, rd, 0, tr < TRW - 1 ? tr + 1 : TRW - 1)[tx];
            const bool mon_plane = MON && J == 1 && zo >= z0 && zo < z1;
            // buffer over output plane zo (used at J == K only): rows at
            // offset kNoStore fall outside it and are not written
            const __amdgpu_buffer_rsrc_t orsrc =
                __builtin_amdgcn_make_buffer_rsrc(out + (J == K ? ooff : 0), (short)0, (int)(PS * 8), kBufWord3);
            // Every row is computed, also the ring rows ry < J and
            // ry >= RH - J, whose values at this level are wrong: they only
            // reach ring rows of the next level and rows that are neither
            // stored nor monitored (oof is kNoStore there), and skipping them
            // would cost a test per row in every wavefront to spare work in
            // the two edge wavefronts, which otherwise wait at the barrier.
            double xi[RYT], th[RYT];  // (compiled root variants: all rows' roots at once)
#pragma unroll
            for (int r = 0; r < RYT; ++r) {
                const double p = cq[r];
                const double zp = zpq[r];
                const double ym = (r > 0) ? cq[r > 0 ? r - 1 : 0] : eT;
                const double yp = (r < RYT - 1) ? cq[r < RYT - 1 ? r + 1 : 0] : eB;
                const double nsum = ((zmq[r] + zp) + (ym + yp)) + (xm[r] + xp[r]);
                if constexpr (RV > 0) {
                    xi[r] = explicit_n<3, RV>(p, nsum, c);
                } else {
                    const double v = update_n<3, RV>(p, nsum, c);
                    if (J < K) dst[r] = v;
                    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(BufB64, v), orsrc, (int)oof[r], 0, 0);
                }
                if (mon_plane && oof[r] != kNoStore) {
                    const double dz = zp - p, dy = yp - p, dx = xp[r] - p;
                    double g = fma(dz, dz, fma(dy, dy, dx * dx));
                    if (BC == BC_HD) {
                        if (zo == 0) g = fma(p, p, g);
                        if (yb0[r]) g = fma(p, p, g);
                        if (xb0) g = fma(p, p, g);
                    }
                    m.bulk += bulk_term(p);
                    m.grad += g;
                    m.mx = nan_max(m.mx, fabs(p));
                }
            }
            if constexpr (RV > 0) {
                cubic_roots_n<RV>(xi, th, c);
#pragma unroll
                for (int r = 0; r < RYT; ++r) {
                    if (J < K) dst[r] = th[r];
                    else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(BufB64, th[r]), orsrc, (int)oof[r], 0, 0);
                }
            }
            if (J < K) {
                const int wr = (int)(zc & 1);
                eb(J, wr, 0, tr)[tx] = dst[0];
                eb(J, wr, 1, tr)[tx] = dst[RYT - 1];
            }
        };

        // One march position with the queue slots fixed at compile time:
        // level 0 planes zc-1, zc, zc+1 in q0[S % 3 ..], level j planes
        // zc-j-1, zc-j, zc-j+1 in qj[j-1][S % 3 ..] (the last written here).
        auto body = [&](auto SS) __attribute__((always_inline)) -> bool {
            constexpr int S = decltype(SS)::value;
            constexpr int P0 = S % 3, P1 = (S + 1) % 3, P2 = (S + 2) % 3;
            // level 1 of plane zc
            level(std::integral_constant<int, 1>(), q0[P0], q0[P1], q0[P2], qj[0][P2]);
            // next level-0 plane into the slot level 1 just freed
            {
                if (zc + 2 <= zlast) cur.next((int)s.M0, PS);  // plane min(zc + 2, zlast)
#pragma unroll
                for (int r = 0; r < RYT; ++r) q0[P0][r] = ld(cur, r);
            }
            // levels 2..K, each from the one below (active once its inputs exist)
            if constexpr (K >= 2) {
                if (zc >= z0 - K + 3)
                    level(std::integral_constant<int, 2>(), qj[0][P0], qj[0][P1], qj[0][P2],
                          qj[K >= 3 ? 1 : 0][P2]);
            }
            if constexpr (K >= 3) {
                if (zc >= z0 - K + 5)
                    level(std::integral_constant<int, 3>(), qj[1][P0], qj[1][P1], qj[1][P2],
                          qj[K >= 4 ? 2 : 1][P2]);
            }
            if constexpr (K >= 4) {
                if (zc >= z0 - K + 7)
                    level(std::integral_constant<int, 4>(), qj[2][P0], qj[2][P1], qj[2][P2], qj[2][P2]);
            }
            if (zc >= zend) return true;
            // edges of level-0 plane zc+1 for the next position
            eb(0, (int)(zc & 1), 0, tr)[tx] = q0[P2][0];
            eb(0, (int)(zc & 1), 1, tr)[tx] = q0[P2][RYT - 1];
            __syncthreads();
            ++zc;
            ooff += PS;
            return false;
        };
        for (;;) {
            if (body(std::integral_constant<int, 0>())) break;
            if (body(std::integral_constant<int, 1>())) break;
            if (body(std::integral_constant<int, 2>())) break;
        }
        __syncthreads();  // every wavefront is done with the edge buffers of this segment
    }
    if (MON) block_reduce_store(m, red, partials + 3 * t);
}

}  // namespace tb3
}  // namespace ace

namespace ace {
namespace tb3 {

// Tile counts of a region shape on the (i1, i2) plane.
template <int K, int TRW, int RYT>
void tiles(const Shape &s, int &tiles_x, int &tiles_y)
{
    using G = Geom<K, TRW, RYT>;
    tiles_x = (int)((s.M2 + G::OX - 1) / G::OX);
    tiles_y = (int)((s.M1 + G::OY - 1) / G::OY);
}

constexpr int64_t PERSIST_MIN = 16;  // least tile-planes per persistent workgroup

template <int K, int TRW, int RYT>
int64_t partials_needed(const Shape &s, int zchunk)
{
    int tx, ty;
    tiles<K, TRW, RYT>(s, tx, ty);
    const int64_t nt = (int64_t)tx * ty;
    if (zchunk <= 0) return std::max<int64_t>(1, std::min<int64_t>(8192, nt * s.M0 / PERSIST_MIN));
    return nt * ((s.M0 + zchunk - 1) / zchunk);
}

// Workgroups of one kernel instance that fit on the device at once (cached
// per device; 0 if the query fails).
template <int BC, bool MON, int RV, int K, int TRW, int RYT, int OCC>
int64_t resident_blocks()
{
    static int64_t cache[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    if (cache[dev] == 0) {
        int per_cu = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_tb3<BC, MON, RV, K, TRW, RYT, OCC>,
                                                         RX * TRW, 0) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 0;
        cache[dev] = (int64_t)std::max(per_cu, 1) * cus;
    }
    return cache[dev];
}

template <int BC, bool MON, int RV, int K, int TRW, int RYT, int OCC>
hipError_t launch(const Shape &s, const StepCoef &c, const double *in, double *out, double *partials,
                  int64_t *nparts, int zchunk, hipStream_t st)
{
    int tiles_x, tiles_y;
    tiles<K, TRW, RYT>(s, tiles_x, tiles_y);
    int64_t nblk;
    if (zchunk > 0) {
        nblk = (int64_t)tiles_x * tiles_y * ((s.M0 + zchunk - 1) / zchunk);
    } else {
        const int64_t res = resident_blocks<BC, MON, RV, K, TRW, RYT, OCC>();
        if (res <= 0) return hipErrorInvalidValue;
        nblk = std::min<int64_t>(res, partials_needed<K, TRW, RYT>(s, 0));
    }
    if (nblk < 1 || nblk > INT32_MAX) return hipErrorInvalidValue;
    if (nparts) *nparts = nblk;
    hipLaunchKernelGGL((k_tb3<BC, MON, RV, K, TRW, RYT, OCC>), dim3((unsigned)nblk), dim3(RX * TRW), 0, st,
                       s, c, in, out, partials, tiles_x, tiles_y, zchunk);
    return hipGetLastError();
}

// Dispatch over the boundary condition, the monitor flag and the root variant.
template <int K, int TRW, int RYT, int OCC>
hipError_t launch_any(const Shape &s, const StepCoef &c, const double *in, double *out,
                      double *partials, int64_t *nparts, int zchunk, hipStream_t st)
{
    auto go = [&](auto BCc, auto RVc) {
        constexpr int B = decltype(BCc)::value, R = decltype(RVc)::value;
        return partials ? launch<B, true, R, K, TRW, RYT, OCC>(s, c, in, out, partials, nparts, zchunk, st)
                        : launch<B, false, R, K, TRW, RYT, OCC>(s, c, in, out, partials, nparts, zchunk, st);
    };
    auto by_rv = [&](auto BCc) {
        return with_root(c.rv, [&](auto RVc) { return go(BCc, RVc); });
    };
    switch (s.bc) {
    case BC_HN: return by_rv(std::integral_constant<int, BC_HN>());
    case BC_HD: return by_rv(std::integral_constant<int, BC_HD>());
    case BC_P: return by_rv(std::integral_constant<int, BC_P>());
    default: return hipErrorInvalidValue;
    }
}

}  // namespace tb3
}  // namespace ace
