// Batches of independent 1D/2D instances.
//
// Three kinds of work, each in launches over all its instances:
//   * 2D instances advance together in rounds of up to `depth` steps over
//     register-resident regions (ace_tb2.h), one launch per round, the fields
//     alternating between the two arenas.  (One workgroup per whole instance
//     left the largest one's time as the launch's: 66 ms for the 1024
//     instances whose rounds take 22.)
//   * 1D instances likewise, one wavefront per segment (ace_tb1.h); those whose
//     indices a segment's 32 bits do not hold (tb1_supported, from about 2^30
//     nodes) by the one-step kernel, a launch per step.
//   * with LDS-plane regions chosen, 2D instances: one workgroup each for all
//     steps, a small field in LDS, others over 32 x 64 LDS regions.
// Every instance carries its own shape, boundary condition, kappa, h and root
// variant, and every update uses the same arithmetic as the single-instance
// kernels, so each instance's result equals ace_step on that instance bit for
// bit.  The launches of 64 rounds are captured once into a HIP graph, which the
// step calls replay; the rest of a call is launched directly.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/ace.h"
#include "ace_device.h"
#include "ace_runtime.h"
#include "ace_tb1.h"
#include "ace_tb2.h"
#include "ace_tile2d.h"

namespace ace {

// How a batch steps an instance of this shape at region rows `region`: all
// its steps by one workgroup, in rounds over 2D regions or 1D segments, or a
// launch per step.
int batch_route(const Shape &s, int region)
{
    if (s.d == 1) return tb1_supported(s) ? BATCH_SEGMENTS : BATCH_STEPS;
    return region != 0 && tb2_supported(s) ? BATCH_REGIONS : BATCH_SINGLE;
}

struct BatchInst {
    int d, bc;
    int64_t M1, M2;   // 1D: 1 x M; 2D: M0 x M1 of the problem
    int64_t total;
    int64_t off;      // field offset in both arenas (doubles)
    StepCoef c;
    int resident;     // 1: stepped in LDS
};

namespace {

constexpr int kBT = 1024;                       // threads per workgroup
constexpr int kBNodes = (int)((RESIDENT_MAX + kBT - 1) / kBT);

// Small 2D instance, the field in LDS for all its steps.
template <int BC, int RV>
__device__ void batch_resident(const BatchInst &I, double *__restrict__ fa, int64_t nsteps, double *f)
{
    const StepCoef c = I.c;
    const int total = (int)I.total;
    const int tid = threadIdx.x;
    const int M1 = (int)I.M1, M2 = (int)I.M2;
    int nb_lo[kBNodes][2], nb_hi[kBNodes][2];
#pragma unroll
    for (int k = 0; k < kBNodes; ++k) {
        const int j = tid + k * kBT;
        const int jj = j < total ? j : 0;
        const int cc[2] = {jj / M2, jj % M2};
        const int n[2] = {M1, M2};
        const int st[2] = {M2, 1};
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            int lo, hi;
            if (cc[a] > 0) lo = j - st[a];
            else lo = (BC == BC_HN) ? j : (BC == BC_HD ? total : j + (n[a] - 1) * st[a]);
            if (cc[a] < n[a] - 1) hi = j + st[a];
            else hi = (BC == BC_HN) ? j : (BC == BC_HD ? total : j - (n[a] - 1) * st[a]);
            nb_lo[k][a] = lo;
            nb_hi[k][a] = hi;
        }
    }
    for (int j = tid; j < total; j += kBT) f[j] = fa[j];
    if (tid == 0) f[total] = 0.0;
    __syncthreads();
    for (int64_t step = 0; step < nsteps; ++step) {
        double nv[kBNodes];
#pragma unroll
        for (int k = 0; k < kBNodes; ++k) {
            const int j = tid + k * kBT;
            nv[k] = 0.0;
            if (j < total) {
                double nsum = 0.0;
#pragma unroll
                for (int a = 0; a < 2; ++a) nsum += f[nb_lo[k][a]] + f[nb_hi[k][a]];
                nv[k] = update_n<2, RV>(f[j], nsum, c);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kBNodes; ++k) {
            const int j = tid + k * kBT;
            if (j < total) f[j] = nv[k];
        }
        __syncthreads();
    }
    for (int j = tid; j < total; j += kBT) fa[j] = f[j];
}

// 2D instance too large for LDS, advanced in rounds of up to tk steps (the
// batch's depth, 1..kMaxDepth): each round walks the instance's 32 x 64
// regions (ring of K nodes), advances each region K levels in LDS (the two
// padded planes live in the workgroup's LDS array) and writes its tile
// interior to the other arena slot; a workgroup barrier (with its memory
// fence) separates the rounds.  The arithmetic and neighbour order are those
// of the single-instance kernels.
constexpr int kMaxDepth = 8;

template <int BC>
__device__ void batch_tiles2d(const BatchInst &I, double *__restrict__ fa, double *__restrict__ fb,
                              int64_t nsteps, double *lds, int tk)
{
    using namespace tile2d;
    constexpr int TR = kBT / BX;  // thread rows
    constexpr int RT = BH / TR;   // region rows per thread
    static_assert(2 * BLP <= RESIDENT_MAX + 1, "two padded planes must fit the LDS array");
    Shape s;
    s.d = 2;
    s.bc = BC;
    s.M0 = 1;
    s.M1 = I.M1;
    s.M2 = I.M2;
    const int tx = threadIdx.x & (BX - 1), tr = threadIdx.x / BX;
    double *F = lds;
    for (int i = threadIdx.x; i < 2 * BLP; i += kBT) F[i] = 0.0;  // zero pads
    __syncthreads();
    int64_t done = 0;
    int par = 0;  // 0: the field is in fa
    while (done < nsteps) {
        const int K = (int)std::min<int64_t>(tk, nsteps - done);
        const double *__restrict__ in = par ? fb : fa;
        double *__restrict__ out = par ? fa : fb;
        const int64_t tiles_x = (s.M2 + BX - 2 * K - 1) / (BX - 2 * K);
        const int64_t tiles_y = (s.M1 + BH - 2 * K - 1) / (BH - 2 * K);
        const int64_t ntiles = tiles_x * tiles_y;
        // the next region's values are loaded into registers while the
        // current region advances, and staged after its last level
        double nxt[RT];
        auto fetch = [&](int64_t t) {
            const Geo gn = make_geo<BC>(s, K, tiles_x, t, tx);
#pragma unroll
            for (int j = 0; j < RT; ++j) {
                const int64_t o = goff<BC>(s, gn.y0r + tr + TR * j, gn.xg);
                nxt[j] = (o < 0) ? 0.0 : in[o];
            }
        };
        fetch(0);
        for (int64_t t = 0; t < ntiles; ++t) {
            const Geo g = make_geo<BC>(s, K, tiles_x, t, tx);
            const bool xin = g.xg >= 0 && g.xg < s.M2 && tx >= K && tx < BX - K;
#pragma unroll
            for (int j = 0; j < RT; ++j) F[(tr + TR * j + 1) * BLW + tx + 1] = nxt[j];
            __syncthreads();
            if (t + 1 < ntiles) fetch(t + 1);
            for (int k = 1; k <= K; ++k) {
                const double *src = F + ((k - 1) & 1) * BLP;
                double *dst = F + (k & 1) * BLP;
#pragma unroll
                for (int j = 0; j < RT; ++j) {
                    const int ry = tr + TR * j;
                    if (ry < k || ry >= BH - k) continue;  // wave-uniform
                    int ym, yp;
                    yoffs<BC>(s, g, ry, ym, yp);
                    const int o = (ry + 1) * BLW + tx + 1;
                    const double p = src[o];
                    const double nsum = (src[o + ym] + src[o + yp]) + (src[o + g.xm] + src[o + g.xp]);
                    const double v = update<2>(p, nsum, I.c);
                    dst[o] = v;
                    const int64_t yg = g.y0r + ry;
                    if (k == K && xin && ry >= K && ry < BH - K && yg >= 0 && yg < s.M1)
                        out[yg * s.M2 + g.xg] = v;
                }
                __syncthreads();
            }
        }
        __threadfence_block();
        __syncthreads();
        done += K;
        par ^= 1;
    }
    if (par) {  // result back into the first arena
        for (int64_t j = threadIdx.x; j < s.M1 * s.M2; j += kBT) fa[j] = fb[j];
        __threadfence_block();
        __syncthreads();
    }
}

// f with the instance's boundary condition and root variant (batches have no
// explicit scheme).
template <class F>
__device__ __forceinline__ void with_instance(const BatchInst &I, F &&f)
{
    auto by_rv = [&](auto BCc) {
        with_root(I.c.rv, [&](auto RVc) {
            constexpr int RV = decltype(RVc)::value;
            f(BCc, RootTag<RV == ROOT_FEX ? 0 : RV>());
        });
    };
    if (I.bc == BC_HN) by_rv(RootTag<BC_HN>());
    else if (I.bc == BC_HD) by_rv(RootTag<BC_HD>());
    else by_rv(RootTag<BC_P>());
}

// One workgroup's piece of a launch over many instances: the instance, and
// its tile row and column (regions), segment or chunk number.
struct Piece {
    int inst, a, b;
};

// One region of a 2D instance per workgroup, S steps from src to dst (a ring
// of K >= S nodes).  Two workgroups fit on a CU, so one's loads overlap the
// other's levels: 225 us per round of 5 steps on 512 instances of 24.5 million
// nodes, where the region levels take 150 and the field's bytes 110 at the
// rate of a copy.  (A persistent grid that loads the next region while it
// advances the current one needs 71 vector registers and spills at the 64 of
// two workgroups: 325 us.)
template <int RYT>
__global__ __launch_bounds__(kBT) void k_batch_regions(const BatchInst *__restrict__ inst,
                                                      const Piece *__restrict__ pieces, const double *__restrict__ src,
                                                      double *__restrict__ dst, int K, int S)
{
    constexpr int TRW = kBT / 64;  // 16 wavefronts
    __shared__ double EB[2 * 2 * TRW * 64];
    const Piece p = pieces[xcd_tile(blockIdx.x, gridDim.x)];
    const BatchInst &I = inst[p.inst];
    with_instance(I, [&](auto BCc, auto RVc) {
        constexpr int RV = decltype(RVc)::value;
        Shape s;
        s.d = 2;
        s.bc = decltype(BCc)::value;
        s.M0 = 1;
        s.M1 = I.M1;
        s.M2 = I.M2;
        MonAcc m;
        mon_zero(m);
        const tb2::Region<decltype(BCc)::value, TRW, RYT> g(s, K, p.a, p.b);
        double v[RYT];
        g.load(s, src + I.off, v);
        g.template advance<false, false, RV>(s, coef_vgpr<RV>(I.c), v, dst + I.off, 0, EB, m, S);
    });
}

// One segment of a 1D instance, S steps from src to dst
// (kSegR nodes per lane, a ring of kSegK >= S nodes on each side).
constexpr int kSegR = 4, kSegK = 32, kSegOut = 64 * kSegR - 2 * kSegK;

__global__ __launch_bounds__(64) void k_batch_segments(const BatchInst *__restrict__ inst,
                                                       const Piece *__restrict__ pieces,
                                                       const double *__restrict__ src, double *__restrict__ dst, int S)
{
    const Piece p = pieces[blockIdx.x];
    const BatchInst &I = inst[p.inst];
    with_instance(I, [&](auto BCc, auto RVc) {
        constexpr int BC = decltype(BCc)::value, RV = decltype(RVc)::value;
        const StepCoef c = coef_vgpr<RV>(I.c);
        const int n = (int)I.total, o0 = p.a * kSegOut, o1 = o0 + kSegOut < n ? o0 + kSegOut : n;
        const int first = o0 - kSegK + (int)threadIdx.x * kSegR;
        double v[kSegR];
#pragma unroll
        for (int r = 0; r < kSegR; ++r) {
            int sg;
            const double x = src[I.off + tb1::source<BC>(first + r, n, sg)];
            v[r] = (BC != BC_HD || sg > 0) ? x : (sg < 0 ? -x : 0.0);
        }
        for (int k = 0; k < S; ++k) tb1::step<kSegR, RV>(v, c);
#pragma unroll
        for (int r = 0; r < kSegR; ++r)
            if (first + r >= o0 && first + r < o1) dst[I.off + first + r] = v[r];
    });
}

// All steps of one 2D instance per workgroup: small ones in LDS, others over
// LDS-plane regions.
__global__ __launch_bounds__(kBT) void k_batch(const BatchInst *__restrict__ inst, const int *__restrict__ order,
                                               double *__restrict__ arena_a, double *__restrict__ arena_b,
                                               int64_t nsteps, int tk)
{
    __shared__ double f[RESIDENT_MAX + 1];
    const BatchInst &I = inst[order[blockIdx.x]];
    double *fa = arena_a + I.off;
    double *fb = arena_b + I.off;
    if (I.resident) {
        with_instance(I, [&](auto BCc, auto RVc) {
            batch_resident<decltype(BCc)::value, decltype(RVc)::value>(I, fa, nsteps, f);
        });
    } else if (I.bc == BC_HN) {
        batch_tiles2d<BC_HN>(I, fa, fb, nsteps, f, tk);
    } else if (I.bc == BC_HD) {
        batch_tiles2d<BC_HD>(I, fa, fb, nsteps, f, tk);
    } else {
        batch_tiles2d<BC_P>(I, fa, fb, nsteps, f, tk);
    }
}

// Chunks of kChunk nodes of every instance, for the copies and the monitor.
constexpr int kChunk = 4096;
constexpr int kChunkThreads = 256;

// dst[...] = src[...] over each chunk: between the arenas (packed = nullptr),
// or from (to_packed) or to the fields back to back in instance order,
// instance i at packed[i].
__global__ __launch_bounds__(kChunkThreads) void k_batch_copy(const BatchInst *__restrict__ inst,
                                                              const Piece *__restrict__ pieces,
                                                              const int64_t *__restrict__ packed, int to_packed,
                                                              const double *__restrict__ src, double *__restrict__ dst)
{
    const Piece p = pieces[blockIdx.x];
    const int64_t off = inst[p.inst].off, total = inst[p.inst].total;
    const int64_t lo = (int64_t)p.a * kChunk, hi = lo + kChunk < total ? lo + kChunk : total;
    const int64_t so = packed && !to_packed ? packed[p.inst] : off, to = packed && to_packed ? packed[p.inst] : off;
#pragma unroll 4
    for (int64_t j = lo + threadIdx.x; j < hi; j += kChunkThreads) dst[to + j] = src[so + j];
}

// Monitor partial (bulk, grad, max) of each chunk.
__global__ __launch_bounds__(kChunkThreads) void k_batch_monitor(const BatchInst *__restrict__ inst,
                                                                 const Piece *__restrict__ pieces,
                                                                 const double *__restrict__ arena_a,
                                                                 double *__restrict__ partials)
{
    __shared__ double lds[3 * (kChunkThreads / 64)];
    const Piece p = pieces[blockIdx.x];
    const BatchInst &I = inst[p.inst];
    const double *f = arena_a + I.off;
    const int64_t lo = (int64_t)p.a * kChunk, hi = lo + kChunk < I.total ? lo + kChunk : I.total;
    const int d = I.d, bc = I.bc;
    const int64_t M1 = I.M1, M2 = I.M2;
    int64_t i1 = (lo + threadIdx.x) / M2, i2 = (lo + threadIdx.x) - i1 * M2;
    MonAcc m;
    mon_zero(m);
    for (int64_t j = lo + threadIdx.x; j < hi; j += kChunkThreads) {
        const double v = f[j];
        double g = 0.0;
        auto axis = [&](int64_t c, int64_t n, int64_t st) {
            double nx;
            if (c < n - 1) nx = f[j + st];
            else nx = (bc == BC_HN) ? v : (bc == BC_HD ? 0.0 : f[j - (n - 1) * st]);
            const double dh = nx - v;
            g = fma(dh, dh, g);
            if (bc == BC_HD && c == 0) g = fma(v, v, g);
        };
        if (d == 2) axis(i1, M1, M2);
        axis(i2, M2, 1);
        m.bulk += bulk_term(v);
        m.grad += g;
        m.mx = nan_max(m.mx, fabs(v));
        i2 += kChunkThreads;
        while (i2 >= M2) {
            i2 -= M2;
            ++i1;
        }
    }
    block_reduce_store(m, lds, partials + 3 * blockIdx.x);
}

// The chunks' partials of instance i (first[i] .. first[i + 1]) in order.
__global__ __launch_bounds__(64) void k_batch_monitor_sum(const int *__restrict__ first,
                                                          const double *__restrict__ partials,
                                                          double *__restrict__ trip)
{
    MonAcc m;
    mon_zero(m);
    for (int j = first[blockIdx.x] + threadIdx.x; j < first[blockIdx.x + 1]; j += 64) {
        m.bulk += partials[3 * (int64_t)j + 0];
        m.grad += partials[3 * (int64_t)j + 1];
        m.mx = nan_max(m.mx, partials[3 * (int64_t)j + 2]);
    }
    const double b = wave_sum(m.bulk), g = wave_sum(m.grad), x = wave_max(m.mx);
    if (threadIdx.x == 0) {
        trip[3 * blockIdx.x + 0] = b;
        trip[3 * blockIdx.x + 1] = g;
        trip[3 * blockIdx.x + 2] = x;
    }
}

}  // namespace
}  // namespace ace

using namespace ace;

struct ace_batch {
    int count = 0;
    std::vector<Problem> prob;
    std::vector<BatchInst> host_inst;
    std::vector<int64_t> packed;  // offsets of the fields back to back
    int64_t arena_total = 0, packed_total = 0;
    int64_t resident_limit = RESIDENT_MAX;  // tuned: largest field stepped in LDS
    int depth = 4;    // steps per round of the large 2D instances (set or tuned, or by rule)
    int depth_fixed = 0;
    int region = 64;  // tuned: 0 LDS-plane 32 x 64 regions; 32 or 64: register-resident regions of that height
    int device = 0;
    hipStream_t stream = nullptr;   // caller's stream (graph launches go here)
    hipStream_t capture = nullptr;  // private stream used only for graph capture
    BatchInst *inst = nullptr;
    int *order_dev = nullptr;
    int64_t *packed_dev = nullptr;
    // pieces of every launch kind, one device array: regions of the 2D
    // instances at the current depth and region, segments of the 1D ones,
    // chunks of all instances (for the copies and the monitor), and those of
    // the instances in regions, in segments and of `by_step`
    Piece *pieces = nullptr;
    int n_regions = 0, n_segments = 0, n_chunks = 0, n_chunks2 = 0, n_chunks1 = 0, n_chunks0 = 0;
    std::vector<int> by_step;  // 1D instances too large for segments
    int *chunk_first = nullptr;  // count + 1
    int n_single = 0;  // order_dev[]: the 2D instances of k_batch
    double *arena_a = nullptr, *arena_b = nullptr;
    double *trip = nullptr, *partials = nullptr;
    int use_graphs = 1;  // 0: the launches are issued directly on every step call
    hipGraph_t graph = nullptr;  // graph_steps() steps at the current choice
    hipGraphExec_t graph_exec = nullptr;
};

namespace {

#define BT_TRY(expr)            \
    do {                        \
        const int _rc = (expr); \
        if (_rc < 0) return _rc; \
    } while (0)
#define BT_HIP(expr) BT_TRY(hip_status(expr))

void drop_graphs(ace_batch *b)
{
    // a replay may still run on the handle's stream
    if (!b->graph_exec) return;
    (void)hipStreamSynchronize(b->stream);
    (void)hipGraphExecDestroy(b->graph_exec);
    (void)hipGraphDestroy(b->graph);
    b->graph_exec = nullptr;
    b->graph = nullptr;
}

// What a batch's launches are made from: the choices, the instances of each
// kind of work and the tables on the device.
struct Choice {
    int64_t resident_limit;
    int depth, depth_fixed, region;
};

Choice choice_of(const ace_batch *b) { return {b->resident_limit, b->depth, b->depth_fixed, b->region}; }

// Sorts the instances into their kinds of work at choice c, uploads the tables
// of the launches, and only then takes both over: on an error the batch keeps
// the choice and the tables it had.
int upload_tables(ace_batch *b, Choice c)
{
    // the tables below are read by any launch still running on the stream
    BT_HIP(hipStreamSynchronize(b->stream));
    std::vector<BatchInst> inst = b->host_inst;
    std::vector<int> large2, large1, single, by_step;
    for (int i = 0; i < b->count; ++i) {
        BatchInst &I = inst[i];
        // (in LDS, a small instance takes longer than as its few regions or
        // segments: 200 of 16^2 to 60^2 and of 128 to 4096 nodes x 500 steps
        // 1.97 against 0.97 ms)
        I.resident = I.d == 2 && c.region == 0 && I.total <= c.resident_limit;
        switch (batch_route(shape_of(b->prob[i]), c.region)) {
        case BATCH_SEGMENTS: large1.push_back(i); break;
        case BATCH_REGIONS: large2.push_back(i); break;
        case BATCH_STEPS: by_step.push_back(i); break;
        default: single.push_back(i);
        }
    }
    // workgroups that take a whole instance: the costly ones first
    std::stable_sort(single.begin(), single.end(), [&](int x, int y) { return inst[x].total > inst[y].total; });
    // regions of one code path (boundary condition, root variant) next to each other
    std::stable_sort(large2.begin(), large2.end(), [&](int x, int y) {
        const BatchInst &X = inst[x], &Y = inst[y];
        return X.bc != Y.bc ? X.bc < Y.bc : X.c.rv < Y.c.rv;
    });
    if (!c.depth_fixed && c.region == 64) {
        // the least modelled time per step: workgroups of the busiest of 256
        // CUs, two of which run together (0.62 us per level alone, 1.1 the
        // two), 3 levels to load and store, and 3.7 us per launch.  On 16
        // batches of 12 to 1024 2D instances the chosen depth was within 2%
        // of the fastest (0.2% on the mean); with 1.2 levels, as for one
        // field, within 10% (4096 instances: 101.3 ms at 4 steps per round,
        // 96.3 at 5).
        double best = 1e300;
        for (int K = 2; K <= kMaxDepth; ++K) {
            int64_t n = 0;
            for (int i : large2) {
                const BatchInst &I = inst[i];
                n += ((I.M1 + 63 - 2 * K) / (64 - 2 * K)) * ((I.M2 + 63 - 2 * K) / (64 - 2 * K));
            }
            const int64_t busiest = (n + 255) / 256;
            const double us = (3.7 + (K + 3) * (1.1 * (double)(busiest / 2) + 0.62 * (double)(busiest % 2))) / K;
            if (us >= best) continue;
            best = us;
            c.depth = K;
        }
    }
    std::vector<Piece> p;
    const int oy = std::max(1, c.region - 2 * c.depth), ox = 64 - 2 * c.depth;
    for (int i : large2) {
        const BatchInst &I = inst[i];
        for (int y = 0; y < (I.M1 + oy - 1) / oy; ++y)
            for (int x = 0; x < (I.M2 + ox - 1) / ox; ++x) p.push_back({i, y, x});
    }
    const size_t n_regions = p.size();
    for (int i : large1)
        for (int64_t a = 0; a * kSegOut < inst[i].total; ++a) p.push_back({i, (int)a, 0});
    const size_t n_segments = p.size() - n_regions;
    auto chunks_of = [&](int i) {
        for (int64_t a = 0; a * kChunk < inst[i].total; ++a) p.push_back({i, (int)a, 0});
    };
    std::vector<int> first(b->count + 1, 0);
    for (int i = 0; i < b->count; ++i) {
        chunks_of(i);
        first[i + 1] = (int)(p.size() - n_regions - n_segments);
    }
    size_t n_of[3], before = p.size();
    const std::vector<int> *kinds[3] = {&large2, &large1, &by_step};
    for (int k = 0; k < 3; ++k) {
        for (int i : *kinds[k]) chunks_of(i);
        n_of[k] = p.size() - before;
        before = p.size();
    }
    if (p.size() > (size_t)INT32_MAX) return ACE_E_NOMEM;
    if (!b->partials) {  // (the chunks do not depend on the choice)
        BT_HIP(hipMalloc((void **)&b->partials, sizeof(double) * 3 * (size_t)first[b->count]));
        BT_HIP(hipMalloc((void **)&b->chunk_first, sizeof(int) * first.size()));
        BT_HIP(hipMemcpy(b->chunk_first, first.data(), sizeof(int) * first.size(), hipMemcpyHostToDevice));
    }
    Piece *pieces = nullptr;
    BT_HIP(hipMalloc((void **)&pieces, sizeof(Piece) * p.size()));
    int rc = hip_status(hipMemcpy(pieces, p.data(), sizeof(Piece) * p.size(), hipMemcpyHostToDevice));
    if (rc >= 0) rc = hip_status(hipMemcpy(b->inst, inst.data(), sizeof(BatchInst) * b->count, hipMemcpyHostToDevice));
    if (rc >= 0 && !single.empty())
        rc = hip_status(hipMemcpy(b->order_dev, single.data(), sizeof(int) * single.size(), hipMemcpyHostToDevice));
    if (rc < 0) {
        (void)hipFree(pieces);
        return rc;
    }
    drop_graphs(b);
    if (b->pieces) (void)hipFree(b->pieces);
    b->pieces = pieces;
    b->n_regions = (int)n_regions;
    b->n_segments = (int)n_segments;
    b->n_chunks = first[b->count];
    b->n_chunks2 = (int)n_of[0];
    b->n_chunks1 = (int)n_of[1];
    b->n_chunks0 = (int)n_of[2];
    b->n_single = (int)single.size();
    b->by_step.swap(by_step);
    b->host_inst.swap(inst);
    b->resident_limit = c.resident_limit;
    b->depth = c.depth;
    b->depth_fixed = c.depth_fixed;
    b->region = c.region;
    return ACE_OK;
}

int choose(ace_batch *b, const Choice &c)
{
    try {
        return upload_tables(b, c);
    } catch (const std::bad_alloc &) {
        return ACE_E_NOMEM;
    }
}

const Piece *chunk_pieces(const ace_batch *b) { return b->pieces + b->n_regions + b->n_segments; }

// f(first, count) for the parts of n workgroups that a launch of `threads`
// each can hold (one, up to billions of nodes).
template <class F>
void in_parts(int64_t n, int threads, F &&f)
{
    const int64_t most = max_blocks(threads);
    for (int64_t i = 0; i < n; i += most) f(i, (unsigned)std::min(most, n - i));
}

// f(steps, from, to) for each of an even number of rounds of at most `most`
// steps (so that the fields end in the arena they began in), of equal length
// to one step; only an odd number of one-step rounds stays odd.  Returns the
// rounds.
template <class F>
int64_t in_rounds(const ace_batch *b, int64_t nsteps, int most, F &&f)
{
    int64_t rounds = (nsteps + most - 1) / most;
    if ((rounds & 1) && rounds < nsteps) ++rounds;
    int64_t done = 0;
    for (int64_t r = 0; r < rounds; ++r) {
        const int64_t upto = nsteps * (r + 1) / rounds;
        f((int)(upto - done), (r & 1) ? b->arena_b : b->arena_a, (r & 1) ? b->arena_a : b->arena_b);
        done = upto;
    }
    return rounds;
}

// Copies the chunks of pieces[0..n): see k_batch_copy.
void copy_chunks(const ace_batch *b, hipStream_t st, const Piece *pieces, int n, const int64_t *packed, int to_packed,
                 const double *src, double *dst)
{
    in_parts(n, kChunkThreads, [&](int64_t first, unsigned m) {
        hipLaunchKernelGGL(k_batch_copy, dim3(m), dim3(kChunkThreads), 0, st, b->inst, pieces + first, packed,
                           to_packed, src, dst);
    });
}

// The rounds of nsteps steps of the instances in regions and in segments.
hipError_t launch_rounds(const ace_batch *b, hipStream_t st, int64_t nsteps)
{
    // the result of an odd number of rounds back into the first arena
    auto copy_back = [&](const Piece *pieces, int n) { copy_chunks(b, st, pieces, n, nullptr, 0, b->arena_b, b->arena_a); };
    if (b->n_regions > 0) {
        auto go = [&](auto kern) {
            return in_rounds(b, nsteps, b->depth, [&](int S, const double *src, double *dst) {
                in_parts(b->n_regions, kBT, [&](int64_t first, unsigned n) {
                    hipLaunchKernelGGL(kern, dim3(n), dim3(kBT), 0, st, b->inst, b->pieces + first, src, dst, b->depth,
                                       S);
                });
            });
        };
        const int64_t rounds = b->region == 64 ? go(k_batch_regions<4>) : go(k_batch_regions<2>);
        if (rounds & 1) copy_back(chunk_pieces(b) + b->n_chunks, b->n_chunks2);
    }
    if (b->n_segments > 0) {
        const int64_t rounds = in_rounds(b, nsteps, kSegK, [&](int S, const double *src, double *dst) {
            in_parts(b->n_segments, 64, [&](int64_t first, unsigned n) {
                hipLaunchKernelGGL(k_batch_segments, dim3(n), dim3(64), 0, st, b->inst,
                                   b->pieces + b->n_regions + first, src, dst, S);
            });
        });
        if (rounds & 1) copy_back(chunk_pieces(b) + b->n_chunks + b->n_chunks2, b->n_chunks1);
    }
    return hipGetLastError();
}

// All nsteps steps of the other instances: a launch per step, or all of them
// in one workgroup's launch.
hipError_t launch_others(const ace_batch *b, hipStream_t st, int64_t nsteps)
{
    for (int i : b->by_step) {
        const BatchInst &I = b->host_inst[i];
        double *in = b->arena_a + I.off, *out = b->arena_b + I.off;
        for (int64_t k = 0; k < nsteps; ++k, std::swap(in, out)) {
            const hipError_t e = launch_step_direct(shape_of(b->prob[i]), I.c, in, out, nullptr, nullptr, st);
            if (e != hipSuccess) return e;
        }
    }
    if (b->n_chunks0 > 0 && (nsteps & 1))
        copy_chunks(b, st, chunk_pieces(b) + b->n_chunks + b->n_chunks2 + b->n_chunks1, b->n_chunks0, nullptr, 0,
                    b->arena_b, b->arena_a);
    in_parts(b->n_single, kBT, [&](int64_t first, unsigned n) {
        hipLaunchKernelGGL(k_batch, dim3(n), dim3(kBT), 0, st, b->inst, b->order_dev + first, b->arena_a, b->arena_b,
                           nsteps, b->depth);
    });
    return hipGetLastError();
}

// Steps of the batch's one graph: 64 rounds of the regions (or of the segments
// where there are no regions), so that its capture costs the same for any
// number of steps a program asks for.
int64_t graph_steps(const ace_batch *b) { return 64 * (int64_t)(b->n_regions > 0 ? b->depth : kSegK); }

int get_graph(ace_batch *b)
{
    if (b->graph_exec) return ACE_OK;
    BT_HIP(hipStreamBeginCapture(b->capture, hipStreamCaptureModeThreadLocal));
    hipError_t le = launch_rounds(b, b->capture, graph_steps(b));
    hipError_t ce = hipStreamEndCapture(b->capture, &b->graph);
    if (le == hipSuccess) le = ce;
    if (le == hipSuccess) le = hipGraphInstantiate(&b->graph_exec, b->graph, nullptr, nullptr, 0);
    if (le != hipSuccess) {
        if (b->graph) (void)hipGraphDestroy(b->graph);
        b->graph = nullptr;
        b->graph_exec = nullptr;
    }
    return hip_status(le);
}

}  // namespace

extern "C" {

int ace_batch_create(int count, const ace_instance_desc *desc, ace_batch **out, int *status)
{
    if (!out || !desc || count < 1) return ACE_E_ARG;
    *out = nullptr;
    ace_batch *b = new (std::nothrow) ace_batch();
    if (!b) return ACE_E_NOMEM;
    b->count = count;
    b->prob.resize(count);
    b->host_inst.resize(count);
    b->packed.resize(count);
    int worst = ACE_OK, warn = ACE_OK;
    int64_t off = 0;
    for (int i = 0; i < count; ++i) {
        const ace_instance_desc &D = desc[i];
        int rc = (D.d == 1 || D.d == 2) ? derive(D.d, D.N, D.L, D.R, D.eps, D.dt, D.bc, b->prob[i])
                                        : ACE_E_ARG;
        if (status) status[i] = rc;
        if (rc < 0 && worst == ACE_OK) worst = rc;
        if (rc > 0) warn = rc;
        if (rc < 0) continue;
        const Problem &p = b->prob[i];
        BatchInst &I = b->host_inst[i];
        I.d = p.d;
        I.bc = p.bc;
        I.M1 = (p.d == 1) ? 1 : p.M[0];
        I.M2 = (p.d == 1) ? p.M[0] : p.M[1];
        I.total = p.total;
        I.off = off;
        I.c = coef_of(p);
        I.resident = 0;
        off += (p.total + 31) / 32 * 32;  // 256-byte aligned fields
        b->packed[i] = b->packed_total;
        b->packed_total += p.total;
    }
    if (worst < 0) {
        delete b;
        return worst;
    }
    b->arena_total = off;
    (void)hipGetDevice(&b->device);
    int rc = ACE_OK;
    auto fail = [&](int r) {
        ace_batch_destroy(b);
        return r;
    };
    if ((rc = hip_status(hipMalloc((void **)&b->arena_a, sizeof(double) * off))) < 0) return fail(rc);
    if ((rc = hip_status(hipMalloc((void **)&b->arena_b, sizeof(double) * off))) < 0) return fail(rc);
    if ((rc = hip_status(hipMemset(b->arena_a, 0, sizeof(double) * off))) < 0) return fail(rc);
    if ((rc = hip_status(hipMalloc((void **)&b->inst, sizeof(BatchInst) * count))) < 0) return fail(rc);
    if ((rc = hip_status(hipMalloc((void **)&b->order_dev, sizeof(int) * count))) < 0) return fail(rc);
    if ((rc = hip_status(hipMalloc((void **)&b->packed_dev, sizeof(int64_t) * count))) < 0) return fail(rc);
    if ((rc = hip_status(hipMemcpy(b->packed_dev, b->packed.data(), sizeof(int64_t) * count,
                                   hipMemcpyHostToDevice))) < 0)
        return fail(rc);
    if ((rc = hip_status(hipMalloc((void **)&b->trip, sizeof(double) * 3 * count))) < 0) return fail(rc);
    if ((rc = hip_status(hipStreamCreateWithFlags(&b->capture, hipStreamNonBlocking))) < 0) return fail(rc);
    if ((rc = choose(b, choice_of(b))) < 0) return fail(rc);
    *out = b;
    return warn;
}

int ace_batch_destroy(ace_batch *b)
{
    if (!b) return ACE_E_ARG;
    drop_graphs(b);
    void *ptrs[] = {b->arena_a, b->arena_b, b->inst,   b->order_dev, b->packed_dev,
                    b->pieces,  b->trip,    b->partials, b->chunk_first};
    for (void *p : ptrs)
        if (p) (void)hipFree(p);
    if (b->capture) (void)hipStreamDestroy(b->capture);
    delete b;
    return ACE_OK;
}

int ace_batch_shape(const ace_batch *b, int i, int64_t M[3], int64_t *total, int64_t *offset)
{
    if (!b || i < 0 || i >= b->count) return ACE_E_ARG;
    const Problem &p = b->prob[i];
    if (M)
        for (int j = 0; j < 3; ++j) M[j] = p.M[j];
    if (total) *total = p.total;
    if (offset) *offset = b->host_inst[i].off;
    return ACE_OK;
}

int ace_batch_set_stream(ace_batch *b, void *st)
{
    if (!b) return ACE_E_ARG;
    if ((hipStream_t)st != b->stream) {
        leave_stream(b->stream, (hipStream_t)st);
        drop_graphs(b);  // a replay on the old stream may still use a captured graph
    }
    b->stream = (hipStream_t)st;
    return ACE_OK;
}

int ace_batch_set_phi0(ace_batch *b, int i, const double *phi0, int where)
{
    if (!b || !phi0 || i < 0 || i >= b->count || (where != ACE_HOST && where != ACE_DEVICE))
        return ACE_E_ARG;
    const BatchInst &I = b->host_inst[i];
    int warn = ACE_OK;
    if (where == ACE_HOST) {
        for (int64_t j = 0; j < I.total; ++j) {
            if (!isfinite(phi0[j])) return ACE_E_NONFINITE;
            if (fabs(phi0[j]) > 1.0) warn = ACE_W_PHI0_GT1;
        }
    }
    BT_HIP(hipMemcpyAsync(b->arena_a + I.off, phi0, sizeof(double) * I.total,
                          where == ACE_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice,
                          b->stream));
    if (where == ACE_HOST) BT_HIP(hipStreamSynchronize(b->stream));
    return warn;
}

int ace_batch_set_all(ace_batch *b, const double *all, int where)
{
    if (!b || !all || (where != ACE_HOST && where != ACE_DEVICE)) return ACE_E_ARG;
    int warn = ACE_OK;
    const double *src = all;
    if (where == ACE_HOST) {
        for (int64_t j = 0; j < b->packed_total; ++j) {
            if (!isfinite(all[j])) return ACE_E_NONFINITE;
            if (fabs(all[j]) > 1.0) warn = ACE_W_PHI0_GT1;
        }
        // one copy into the second arena (scratch between steps), spread out from there
        BT_HIP(hipMemcpyAsync(b->arena_b, all, sizeof(double) * b->packed_total, hipMemcpyHostToDevice, b->stream));
        src = b->arena_b;
    }
    copy_chunks(b, b->stream, chunk_pieces(b), b->n_chunks, b->packed_dev, 0, src, b->arena_a);
    BT_HIP(hipGetLastError());
    if (where == ACE_HOST) BT_HIP(hipStreamSynchronize(b->stream));
    return warn;
}

int ace_batch_step(ace_batch *b, int64_t nsteps)
{
    if (!b || nsteps < 0) return ACE_E_ARG;
    if (nsteps == 0) return ACE_OK;
    if (b->n_regions + b->n_segments > 0) {
        // (a rest of one step would be an odd round and need a copy back)
        const int64_t P = graph_steps(b);
        int64_t left = nsteps;
        for (; b->use_graphs && left >= P && left != P + 1; left -= P) {
            BT_TRY(get_graph(b));
            BT_HIP(hipGraphLaunch(b->graph_exec, b->stream));
        }
        if (left > 0) BT_HIP(launch_rounds(b, b->stream, left));
    }
    BT_HIP(launch_others(b, b->stream, nsteps));
    return ACE_OK;
}

int ace_batch_set_region(ace_batch *b, int rows)
{
    if (!b || (rows != 0 && rows != 32 && rows != 64)) return ACE_E_ARG;
    if (rows == b->region) return ACE_OK;
    Choice c = choice_of(b);
    c.region = rows;
    return choose(b, c);
}

int ace_batch_set_graphs(ace_batch *b, int enable)
{
    if (!b || (enable != 0 && enable != 1)) return ACE_E_ARG;
    b->use_graphs = enable;
    return ACE_OK;
}

int ace_batch_monitor(ace_batch *b, double *E, double *maxn)
{
    if (!b || !E || !maxn) return ACE_E_ARG;
    in_parts(b->n_chunks, kChunkThreads, [&](int64_t first, unsigned n) {
        hipLaunchKernelGGL(k_batch_monitor, dim3(n), dim3(kChunkThreads), 0, b->stream, b->inst,
                           chunk_pieces(b) + first, b->arena_a, b->partials + 3 * first);
    });
    in_parts(b->count, 64, [&](int64_t first, unsigned n) {
        hipLaunchKernelGGL(k_batch_monitor_sum, dim3(n), dim3(64), 0, b->stream, b->chunk_first + first, b->partials,
                           b->trip + 3 * first);
    });
    BT_HIP(hipGetLastError());
    std::vector<double> t(3 * (size_t)b->count);
    BT_HIP(hipMemcpyAsync(t.data(), b->trip, sizeof(double) * t.size(), hipMemcpyDeviceToHost,
                          b->stream));
    BT_HIP(hipStreamSynchronize(b->stream));
    int rc = ACE_OK;
    for (int i = 0; i < b->count; ++i) {
        E[i] = energy_from(b->prob[i], &t[3 * i]);
        maxn[i] = t[3 * i + 2];
        if (!isfinite(E[i]) || !isfinite(maxn[i])) rc = ACE_E_NONFINITE;
    }
    return rc;
}

int ace_batch_get_phi(ace_batch *b, int i, double *out, int where)
{
    if (!b || !out || i < 0 || i >= b->count || (where != ACE_HOST && where != ACE_DEVICE))
        return ACE_E_ARG;
    const BatchInst &I = b->host_inst[i];
    BT_HIP(hipMemcpyAsync(out, b->arena_a + I.off, sizeof(double) * I.total,
                          where == ACE_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice,
                          b->stream));
    if (where == ACE_HOST) BT_HIP(hipStreamSynchronize(b->stream));
    return ACE_OK;
}

int ace_batch_get_all(ace_batch *b, double *out, int where)
{
    if (!b || !out || (where != ACE_HOST && where != ACE_DEVICE)) return ACE_E_ARG;
    // gathered back to back: in the caller's memory, or in the second arena for one copy to the host
    double *dst = where == ACE_DEVICE ? out : b->arena_b;
    copy_chunks(b, b->stream, chunk_pieces(b), b->n_chunks, b->packed_dev, 1, b->arena_a, dst);
    BT_HIP(hipGetLastError());
    if (where == ACE_HOST) {
        BT_HIP(hipMemcpyAsync(out, dst, sizeof(double) * b->packed_total, hipMemcpyDeviceToHost, b->stream));
        BT_HIP(hipStreamSynchronize(b->stream));
    }
    return ACE_OK;
}

int ace_batch_set_resident_limit(ace_batch *b, int64_t limit)
{
    if (!b || limit < 0) return ACE_E_ARG;
    Choice c = choice_of(b);
    c.resident_limit = std::min<int64_t>(limit, RESIDENT_MAX);
    return choose(b, c);
}

int ace_batch_set_depth(ace_batch *b, int depth)
{
    if (!b || depth < 1 || depth > kMaxDepth) return ACE_E_ARG;
    Choice c = choice_of(b);
    c.depth = depth;
    c.depth_fixed = 1;
    if (depth != b->depth) return choose(b, c);
    b->depth_fixed = 1;
    return ACE_OK;
}

int ace_batch_autotune(ace_batch *b, int64_t trial_steps, char *json, size_t cap)
{
    if (!b || trial_steps < 1) return ACE_E_ARG;
    // keep the current fields: time each candidate on a copy, then restore
    double *save = nullptr;
    BT_HIP(hipMalloc((void **)&save, sizeof(double) * b->arena_total));
    auto restore = [&]() {
        return hip_status(hipMemcpyAsync(b->arena_a, save, sizeof(double) * b->arena_total,
                                         hipMemcpyDeviceToDevice, b->stream));
    };
    int rc = hip_status(hipMemcpyAsync(save, b->arena_a, sizeof(double) * b->arena_total,
                                       hipMemcpyDeviceToDevice, b->stream));
    const bool started = rc >= 0;  // the fields are saved
    const Choice before = choice_of(b);
    // First the region shape and depth of the region rounds at the current
    // resident limit, then, if whole instances per workgroup won (nothing else
    // reads it), the resident limit.  The rule's own depth is among the trials
    // also where it is beyond the others.
    std::vector<std::pair<int, int>> shapes = {{0, 4}};  // (a whole instance per workgroup: only where all are small)
    for (int region : {32, 64})
        for (int depth = 2; depth <= 6; ++depth) shapes.push_back({region, depth});
    if (!before.depth_fixed && before.region == 64 && before.depth > 6) shapes.push_back({64, before.depth});
    const int64_t limits[] = {0, 1024, 2048, 4096, RESIDENT_MAX};
    double best_ms = 1e300;
    int64_t best_lim = b->resident_limit;
    int best_depth = b->depth;
    int best_region = b->region;
    std::string rec = "{\"kind\": \"batch\", \"trial_steps\": " + std::to_string(trial_steps) +
                      ", \"instances\": " + std::to_string(b->count) + ", \"candidates\": [";
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (rc >= 0) rc = hip_status(hipEventCreate(&e0));
    if (rc >= 0) rc = hip_status(hipEventCreate(&e1));
    bool first = true;
    // times one batch step of trial_steps for (lim, depth, region); returns ms or a negative error
    auto trial = [&](int64_t lim, int depth, int region, double *ms_out) -> int {
        int r;
        if ((r = choose(b, {lim, depth, 1, region})) < 0) return r;
        if ((r = restore()) < 0) return r;
        if ((r = ace_batch_step(b, trial_steps)) < 0) return r;  // builds the graph, warms up
        if ((r = restore()) < 0) return r;
        if ((r = hip_status(hipEventRecord(e0, b->stream))) < 0) return r;
        if ((r = ace_batch_step(b, trial_steps)) < 0) return r;
        if ((r = hip_status(hipEventRecord(e1, b->stream))) < 0) return r;
        if ((r = hip_status(hipEventSynchronize(e1))) < 0) return r;
        float ms = 0.f;
        if ((r = hip_status(hipEventElapsedTime(&ms, e0, e1))) < 0) return r;
        *ms_out = ms;
        char buf[160];
        snprintf(buf, sizeof buf, "%s{\"resident_limit\": %lld, \"depth\": %d, \"region\": %d, \"ms\": %.4f}",
                 first ? "" : ", ", (long long)lim, depth, region, ms);
        rec += buf;
        first = false;
        return ACE_OK;
    };
    const int64_t lim0 = b->resident_limit;
    for (const auto &[region, depth] : shapes) {
        if (rc < 0) break;
        double ms = 0.0;
        if ((rc = trial(lim0, depth, region, &ms)) < 0) break;
        if (ms < best_ms) {
            best_ms = ms;
            best_depth = depth;
            best_region = region;
        }
    }
    for (int64_t lim : limits) {
        if (rc < 0 || best_region != 0) break;
        if (lim == lim0) continue;  // timed above
        double ms = 0.0;
        if ((rc = trial(lim, best_depth, best_region, &ms)) < 0) break;
        if (ms < best_ms) {
            best_ms = ms;
            best_lim = lim;
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    // (an error in a trial leaves the fields and the choice as they were)
    if (rc >= 0) rc = choose(b, {best_lim, best_depth, 1, best_region});
    else if (started) (void)choose(b, before);
    const int rr = started ? restore() : ACE_OK;
    if (rc >= 0) rc = rr;
    if (rc >= 0) rc = hip_status(hipStreamSynchronize(b->stream));
    (void)hipFree(save);
    if (rc < 0) return rc;
    rec += "], \"choice\": {\"resident_limit\": " + std::to_string(best_lim) +
           ", \"depth\": " + std::to_string(best_depth) + ", \"region\": " + std::to_string(best_region) + "}}";
    if (log_enabled())
        fprintf(stderr,
                "[ace] batch autotune (%d instances): LDS limit %lld nodes, region depth %d, region rows %d, "
                "%.4f ms\n",
                b->count, (long long)best_lim, best_depth, best_region, best_ms);
    if (json && cap > 0) snprintf(json, cap, "%s", rec.c_str());
    return ACE_OK;
}

}  // extern "C"
