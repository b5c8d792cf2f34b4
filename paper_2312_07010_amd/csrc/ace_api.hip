// Host runtime behind the C ABI declared in include/ace.h: argument checks,
// derived parameters (Sec. 2; Theorem 2 of Sec. 3.2), device buffers, kernel
// dispatch, monitored runs, and the checkpointed reverse sweep.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/ace.h"
#include "ace_internal.h"
#include "ace_runtime.h"

using namespace ace;

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

namespace ace {

bool log_enabled()
{
    static const bool on = getenv("ACE_LOG") != nullptr;
    return on;
}

int hip_status(hipError_t e)
{
    if (e == hipSuccess) return ACE_OK;
    if (e == hipErrorOutOfMemory) return ACE_E_NOMEM;
    if (log_enabled()) fprintf(stderr, "[ace] HIP error: %s\n", hipGetErrorString(e));
    return ACE_E_HIP;
}

int64_t nodes_per_axis(int64_t N, int bc)
{
    if (bc == ACE_BC_HN) return N + 2;
    if (bc == ACE_BC_HD) return N - 1;
    return N;
}

namespace {

using Real = long double;

Real newton(Real x, Real a, Real H)
{
    return x - (x + H * (x * x * x - x) - a) / (1.0L + H * (3.0L * x * x - 1.0L));
}

// The root for xi = a by Newton's method from x, to the last place.  (For
// h > 1/2 the slope near 0 is small and the last places may not settle: there
// until the iteration repeats itself, which newton_steps then does too.)
Real root_from(Real x, Real a, Real H)
{
    const Real tol = H > 0.5L ? 0.0L : 0x1p-63L;
    for (int k = 0; k < 200; ++k) {
        const Real nx = newton(x, a, H);
        if (fabsl(nx - x) <= tol * nx) return nx;
        x = nx;
    }
    return x;
}

// Newton steps from x until it is within 2^-60 of the root th.
int newton_steps(Real x, Real a, Real th, Real H)
{
    int k = 0;
    for (; fabsl(x - th) > 0x1p-60L * th && k < 60; ++k) x = newton(x, a, H);
    return k;
}

// Coefficients (lowest power of w first) of the polynomial S of degree D that
// interpolates (theta - a) / (a w), a = sqrt(1 - w), theta the root for
// xi = a, at D + 1 points of w in (0, 1]: the zeros, but for w = 0, of the
// Chebyshev polynomial of degree D + 2 on the interval that ends at 1 and puts
// its lowest zero at w = 0.  S's error enters theta times w, and that product
// has the zero at w = 0 too, so its largest value over [0, 1] is near the
// least possible.
void root_polynomial(Real H, int D, Real *p)
{
    const Real pi = 3.14159265358979323846264L;
    Real node[ROOT_MAX_DEG + 1], c[ROOT_MAX_DEG + 1];
    const Real c0 = cosl(pi / (2 * (D + 2)));
    for (int j = 0; j <= D; ++j) {
        const Real w = (cosl(pi * (2 * j + 1) / (2 * (D + 2))) + c0) / (1.0L + c0);
        const Real a = sqrtl(1.0L - w);
        node[j] = w;
        c[j] = (root_from(a, a, H) - a) / (a * w);
    }
    for (int k = 1; k <= D; ++k)  // divided differences
        for (int j = D; j >= k; --j) c[j] = (c[j] - c[j - 1]) / (node[j] - node[j - k]);
    p[0] = c[D];
    for (int j = D - 1; j >= 0; --j) {  // p = p (w - node[j]) + c[j]
        p[D - j] = p[D - j - 1];
        for (int k = D - j - 1; k >= 1; --k) p[k] = p[k - 1] - node[j] * p[k];
        p[0] = c[j] - node[j] * p[0];
    }
}

}  // namespace

// The device root's choice for p.h (ace_device.h), for 0 < xi <= 1.
//
// nit and start2: the Newton steps of root_common without a polynomial.  Both
// starts (theta_0 = a + h a (1 - a^2), or to second order in h; theta_0 = a
// for h > 1/2) and the same Newton step are run in long double on a grid of
// a in (0, 1]; nit is the first step count whose largest relative error
// against the converged root is below 2^-60 (well under half an ulp, leaving
// room for the reciprocal estimate and the rounding of the double iteration).
// The second-order start costs two FMAs more and is used where it saves
// steps.
//
// rv and q: the first of the polynomial variants that stays within 2^-60 of
// the root over every eighth point of that grid and a few near 0, or 0 (from
// about dt = 0.45 none does).
void choose_root(Problem &p)
{
    constexpr int G = 2048, NG = G + 8;
    const Real H = p.h;
    Real a[NG + 8], th[NG + 8];
    int need[2] = {1, 1};
    for (int j = 1; j <= NG; ++j) {
        a[j - 1] = (j <= G) ? (Real)j / G : 1.0L - ldexpl(1.0L, -(j - G) * 6);
        // (the root's slope is near 1, so the last point's root plus the step in a is a close start)
        th[j - 1] = root_from(H <= 0.5L && j > 1 && j <= G ? th[j - 2] + 1.0L / G : a[j - 1], a[j - 1], H);
        const Real x = a[j - 1], f = x * x * x - x;
        const Real x1 = H <= 0.5L ? x - H * f : x;
        const Real x2 = H <= 0.5L ? x - H * f * (1.0L - H * (3.0L * x * x - 1.0L)) : x;
        need[0] = std::max(need[0], newton_steps(x1, x, th[j - 1], H));
        need[1] = std::max(need[1], newton_steps(x2, x, th[j - 1], H));
    }
    p.start2 = need[1] < need[0];
    p.nit = need[p.start2];
    for (int j = 0; j < 8; ++j) {
        a[NG + j] = ldexpl(1.0L, -12 - 4 * j);
        th[NG + j] = root_from(a[NG + j], a[NG + j], H);
    }
    auto within = [&](int v, const Real *q) {
        for (int j = 7; j < NG + 8; j += j < G - 1 ? 8 : 1) {
            const Real w = 1.0L - a[j] * a[j];
            Real s = q[ROOT_DEG[v]];
            for (int k = ROOT_DEG[v] - 1; k >= 0; --k) s = s * w + q[k];
            Real x = a[j] + a[j] * w * s;
            for (int k = 0; k < ROOT_NEWTON[v]; ++k) x = newton(x, a[j], H);
            if (!(fabsl(x - th[j]) <= 0x1p-60L * th[j])) return false;
        }
        return true;
    };
    p.rv = 0;
    for (int v = 1; v <= ROOT_POLYS && p.h <= 0.3; ++v) {
        Real q[ROOT_MAX_DEG + 1];
        root_polynomial(H, ROOT_DEG[v], q);
        if (!within(v, q)) continue;
        p.rv = v;
        for (int k = 0; k <= ROOT_DEG[v]; ++k) p.q[k] = (double)q[k];
        break;
    }
}

// Theorem 2's step condition dt <= 1 - 2 d kappa, 0 < kappa < 1/(2d) (with
// 1e-12 relative slack for the equality case); for the explicit comparison
// scheme Remark 2's dt <= (1 - 2 d kappa)/2.
void set_conditions(Problem &p)
{
    double bound = 1.0 - 2.0 * p.d * p.kappa;
    if (p.scheme == ACE_SCHEME_FEX) bound *= 0.5;
    p.cond_ok = (p.dt <= bound * (1.0 + 1e-12)) && p.kappa > 0.0 && p.kappa < 1.0 / (2.0 * p.d);
}

// Validates the ace_create arguments and fills the derived parameters.
int derive(int d, const int64_t *N, const double *L, const double *R, double eps, double dt,
           int bc, Problem &p)
{
    if (!N || !L || !R) return ACE_E_ARG;
    if (d < 1 || d > 3) return ACE_E_ARG;
    if (bc != ACE_BC_HN && bc != ACE_BC_HD && bc != ACE_BC_P) return ACE_E_ARG;
    if (!(eps > 0.0) || !isfinite(eps)) return ACE_E_ARG;
    if (!isfinite(dt)) return ACE_E_ARG;
    const int64_t minN = (bc == ACE_BC_HN) ? 1 : (bc == ACE_BC_HD ? 2 : 3);
    memset(&p, 0, sizeof(p));
    p.d = d;
    p.bc = bc;
    for (int j = 0; j < 3; ++j) {
        p.N[j] = 1;
        p.M[j] = 1;
        p.L[j] = 0.0;
        p.R[j] = 1.0;
    }
    double dx0 = 0.0;
    for (int j = 0; j < d; ++j) {
        if (!isfinite(L[j]) || !isfinite(R[j]) || !(L[j] < R[j])) return ACE_E_ARG;
        if (N[j] < minN) return ACE_E_SIZE;
        if (N[j] > (int64_t)1 << 31) return ACE_E_SIZE;
        const double dx = (R[j] - L[j]) / (double)N[j];
        if (j == 0) dx0 = dx;
        else if (fabs(dx - dx0) > 1e-12 * dx0) return ACE_E_ANISO;
        p.N[j] = N[j];
        p.L[j] = L[j];
        p.R[j] = R[j];
    }
    if (!(dt > 0.0) || !(dt < 2.0)) return ACE_E_DT;
    p.dx = dx0;
    p.dt = dt;
    p.eps = eps;
    // kappa = eps^2 dt / dx^2 (Sec. 2: eps^2 = (omega_1/s) dx^2 / dt)
    p.kappa = eps * eps * dt / (dx0 * dx0);
    p.h = 0.5 * dt;
    // stored nodes: fastest axis last; a d-dimensional field occupies the
    // last d of the three internal axes
    int64_t total = 1;
    for (int j = 0; j < d; ++j) {
        const int64_t m = nodes_per_axis(N[j], bc);
        p.M[j] = m;
        total *= m;
    }
    p.total = total;
    choose_root(p);
    p.scheme = ACE_SCHEME_RLB_MIE;
    set_conditions(p);
    return p.cond_ok ? ACE_OK : ACE_W_CONDITIONS;
}

Shape shape_of(const Problem &p)
{
    Shape s;
    s.d = p.d;
    s.bc = p.bc;
    if (p.d == 1) {
        s.M0 = 1;
        s.M1 = 1;
        s.M2 = p.M[0];
    } else if (p.d == 2) {
        s.M0 = 1;
        s.M1 = p.M[0];
        s.M2 = p.M[1];
    } else {
        s.M0 = p.M[0];
        s.M1 = p.M[1];
        s.M2 = p.M[2];
    }
    return s;
}

StepCoef coef_of(const Problem &p)
{
    StepCoef c;
    c.kappa = p.kappa;
    c.h = p.h;
    c.omh = 1.0 - p.h;
    c.oph = 1.0 + p.h;
    c.h3 = 3.0 * p.h;
    c.hs = p.h > 0.5 ? 0.0 : p.h;
    c.nit = p.nit;
    c.start2 = p.start2;
    c.fex = (p.scheme == ACE_SCHEME_FEX) ? 1 : 0;
    c.rv = c.fex ? ROOT_FEX : p.rv;
    c.dt = p.dt;
    memcpy(c.q, p.q, sizeof c.q);
    return c;
}

void energy_coefs(const Problem &p, double *dxd, double *cg)
{
    *dxd = pow(p.dx, p.d);
    *cg = p.kappa / (2.0 * p.dt);
}

double energy_from(const Problem &p, const double *trip)
{
    // E = dx^d [ sum (phi^2-1)^2/4 + kappa/(2 dt) sum_edges (dphi)^2 ]
    double dxd, cg;
    energy_coefs(p, &dxd, &cg);
    return dxd * (trip[0] + cg * trip[1]);
}

static bool capturing(hipStream_t stream)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &st) == hipSuccess) return st != hipStreamCaptureStatusNone;
    (void)hipGetLastError();  // (the default stream while another one captures)
    return true;
}

void leave_stream(hipStream_t old, hipStream_t next)
{
    if (capturing(next) || capturing(old)) return;
    if (hipStreamSynchronize(old) != hipSuccess) (void)hipGetLastError();
}

int grow(double **ptr, int64_t *cap, int64_t need)
{
    if (*cap >= need && *ptr) return ACE_OK;
    if (*ptr) (void)hipFree(*ptr);
    *ptr = nullptr;
    *cap = 0;
    hipError_t e = hipMalloc((void **)ptr, (size_t)need * sizeof(double));
    if (e != hipSuccess) {
        *ptr = nullptr;
        return hip_status(e);
    }
    *cap = need;
    return ACE_OK;
}

}  // namespace ace

// ---------------------------------------------------------------------------
// allocation-free monitor: device scratch held in a static array
// ---------------------------------------------------------------------------

namespace {

// Doubles of the static scratch: the reduced triple (kTripSlot doubles, so
// the partials that follow stay 256-byte aligned) and up to kNoAllocParts
// partial triples, 1.5 MiB per device for the life of the process.
constexpr int64_t kTripSlot = 32;
constexpr int64_t kNoAllocParts = 65536;
constexpr int64_t kNoAllocDoubles = kTripSlot + 3 * kNoAllocParts;
constexpr int kMaxDevices = 64;

static __device__ __align__(256) double scratch[kNoAllocDoubles];

// Device address of `scratch` on each device (host code must not pass the
// array's name: on the host it is only a stand-in for the symbol).
double *g_scratch[kMaxDevices] = {};
std::mutex g_scratch_mu;

// Looks up the scratch address of the current device once; called by
// ace_create with the handle's device current.
void scratch_setup(int dev)
{
    if (dev < 0 || dev >= kMaxDevices) return;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch[dev]) return;
    void *ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) {
        (void)hipGetLastError();  // leave no error behind for later launches
        if (log_enabled())
            fprintf(stderr, "[ace] scratch lookup on device %d failed: %s\n", dev, hipGetErrorString(e));
        return;
    }
    g_scratch[dev] = (double *)ptr;
}

double *scratch_of(int dev)
{
    if (dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch[dev];
}

}  // namespace

#define ACE_TRY(expr)                  \
    do {                               \
        const int _rc = (expr);        \
        if (_rc < 0) return _rc;       \
    } while (0)
#define ACE_HIP(expr) ACE_TRY(hip_status(expr))

// ---------------------------------------------------------------------------
// solver handle
// ---------------------------------------------------------------------------

// 1D: nodes per lane and steps per launch (or per exchange).
struct Shape1 {
    int R = 1, K = 8;
    double ns = 1e300;  // modelled time per step
};

struct ace_solver {
    Problem p;
    Shape shape;
    StepCoef coef;
    int device = 0;
    hipStream_t stream = nullptr;
    double *own[2] = {nullptr, nullptr};
    double *buf[2] = {nullptr, nullptr};
    int cur = 0;
    double *partials = nullptr;
    int64_t partials_cap = 0;
    double *mon = nullptr;  // device monitor triples
    int64_t mon_cap = 0;
    double *monparts = nullptr;  // partials of several monitors of a monitored run
    int64_t monparts_cap = 0;
    double *pinned = nullptr;  // host pinned scratch (64 doubles, kernels may write it)
    int64_t steps = 0;
    int warn_mask = 0;  // warnings of the last monitored run (ACE_WARN_BIT)
    int kernel = ACE_KERNEL_AUTO;
    int depth = 0;
    int zchunk = 32;  // planes per workgroup of the 3D temporal-blocking kernel (0: persistent)
    int zchunk_fixed = 0;  // 1: zchunk was set or tuned; 0: it follows the variant (tb3_chunks)
    int depth2 = 5;   // steps per launch of the 2D temporal-blocking kernel
    int tb3 = -1;     // variant of the configurable 3D blocked kernel (-1: the two-step kernel)
    int tb2 = -1;     // variant of the register-resident 2D blocked kernel (-1: the LDS-plane kernel)
    struct Tail {
        int v = -1, zchunk = 0;
    } tail[5];  // 3D: variant and plane chunk of a rest of [i] steps shorter than the handle's depth
    Shape1 tb1, res1;  // 1D: the blocked and the one-workgroup kernel's shapes
    int rule_kernel = ACE_KERNEL_DIRECT;  // ACE_KERNEL_AUTO without an autotuned choice
    int plan_fixed = 0;  // 1: a kernel, region or depth was set or tuned, the rule no longer applies
    int tuned_kernel = 0;  // autotuned choice for ACE_KERNEL_AUTO (0: none)
    // reverse mode
    double *ckpt = nullptr;
    int64_t ckpt_cap = 0;
    int64_t ck_every = 0, ck_steps = 0, ck_count = 0;
    int64_t ck_field_version = -1;
    int64_t ck_generation = 0;  // incremented by every ace_forward_ckpt
    double *seg = nullptr;  // two segment buffers, (every + 1) states each
    int64_t seg_cap = 0;
    hipStream_t aux = nullptr;  // recompute stream of the pipelined reverse sweep
    hipEvent_t ev_start = nullptr, ev_rec[2] = {nullptr, nullptr}, ev_rev[2] = {nullptr, nullptr};
    double *lam = nullptr;
    int64_t lam_cap = 0;
    double *gpart = nullptr;
    int64_t gpart_cap = 0;
    double *gsum = nullptr;
    int64_t field_version = 0;
    // graph replay of runs of launches (0 disables)
    int64_t graph_launches = 32;
    hipStream_t capture = nullptr;
    struct GraphEntry {
        int kernel, zchunk, depth2, tb3, tb2, cur;
        const double *b0, *b1;
        hipGraph_t g;
        hipGraphExec_t e;
    };
    std::vector<GraphEntry> graphs;
};

namespace {

// ---------------------------------------------------------------------------
// Launch shape as a rule of the field's size (no timing).  Every choice gives
// the same result bit for bit; ace_autotune measures instead.
// ---------------------------------------------------------------------------

// Modelled time (us) of one launch of a blocked kernel: the workgroups of the
// busiest of 256 CUs, in rounds of those that fit on it together, each round
// `n` march positions (3D) or levels (2D) and `fill` more to start, at the
// time of one measured with one workgroup alone on its CU and with two.
struct BlockModel {
    int per_cu;
    double one, two, fill, launch;
    double us(int64_t workgroups, double n) const
    {
        const int64_t busiest = (workgroups + 255) / 256;
        const int64_t rounds = busiest / per_cu, rest = busiest % per_cu;
        return launch + (n + fill) * ((double)rounds * (per_cu == 2 ? two : one) + (rest ? one : 0.0));
    }
};

// k_tb3: fitted to launches of 64^3 to 512^3 fields at 16 plane chunks.  On 14
// fields at dt <= 0.02 the five best chunks of each variant took 3 to 11% off
// the model on the mean, and the rule's choice at most 11% more than the
// fastest.  The root is not in the model: at dt = 0.1 and 0.2 (a Newton step)
// launches take 40 to 50% more than it says, all variants alike, so the choice
// stays within 3%.  (profiles/launch_models.txt)
constexpr BlockModel TB3_MODEL[TB3_VARIANTS] = {{2, 0.93, 1.68, 1.7, 3.6}, {1, 1.78, 0, 2.7, 0.2}, {1, 1.84, 0, 2.1, 0.2},
                                                {1, 1.33, 0, 2.6, 2.0},    {2, 1.61, 3.23, 0.1, 1.7}, {1, 1.63, 0, 1.0, 2.3},
                                                {1, 2.19, 0, 1.5, 2.3}};
constexpr int TB3_CHUNKS[] = {8, 10, 12, 14, 16, 20, 24, 28, 32, 40, 48, 64, 80, 96, 128, 176, 256, 352, 512};

// Modelled us per step of variant v at plane chunk zc: the larger of the
// march and, on fields past the caches (20 million nodes), 18 bytes of HBM
// per node and launch at 4.6 TB/s; a tenth of the march orders ties.  The
// explicit scheme has a quarter fewer instructions.
double tb3_us(int v, const Shape &s, int zc, bool fex)
{
    const int K = TB3_TABLE[v].depth;
    const double march = TB3_MODEL[v].us(tb3_partials_needed(v, s, zc),
                                         std::min<double>(zc, (double)s.M0) + 2 * K - 2) * (fex ? 0.8 : 1.0);
    const double nodes = (double)s.M0 * (double)s.M1 * (double)s.M2;
    const double hbm = nodes > 2e7 ? nodes * 18.0 / 4.6e6 : 0.0;
    return (std::max(march, hbm) + 0.1 * march) / K;
}

// Plane chunks of variant v that one launch can hold, the least modelled time
// first (none: a plane has too many tiles).
std::vector<int> tb3_chunks(int v, const Shape &s, bool fex)
{
    const int64_t most = max_blocks(64 * TB3_TABLE[v].rows / TB3_TABLE[v].rpt);
    std::vector<std::pair<double, int>> t;
    for (int zc : TB3_CHUNKS)
        if (zc <= std::max<int64_t>(s.M0, 8) && tb3_partials_needed(v, s, zc) <= most)
            t.push_back({tb3_us(v, s, zc, fex), zc});
    std::stable_sort(t.begin(), t.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    std::vector<int> out;
    for (const auto &x : t) out.push_back(x.second);
    return out;
}

// One step of a 3D field: the column kernel (its time is 2.4 us and 16 bytes
// per node from the caches at 4.4 TB/s: 5.9 us at 96^3, 10.8 at 130^3, 16 at
// 160^3), or past 20 million nodes, where the marching kernel reads each
// plane of HBM once, that one (232 against 324 us at 400^3, 430 against 667
// at 512^3; 72 against 58 at 256^3).
constexpr double kColumnUs = 2.4, kColumnUsPerNode = 3.6e-6;

int one_step_kernel(const Shape &s)
{
    if (s.d == 3 && march_supported(s) && s.M0 * s.M1 * s.M2 > 20000000) return ACE_KERNEL_MARCH;
    return ACE_KERNEL_DIRECT;
}

// k_tb2: fitted to 19 fields from 30 x 30 to 3000 x 3000 at depths 2 to 12; a
// level of the 32-row regions is bound by the rows of one CU (0.28 us), so
// small fields take the deepest launch.  All shapes and depths deviate 3 to 10%
// on the mean at dt <= 0.02.  The root is not in the model: at dt = 0.2 (a
// Newton step) 401 x 283 takes 0.94 us per step for 0.69 modelled, 512^2 1.45
// for 0.97, 1024^2 2.81 for 1.90.  The choice was the fastest shape on 14 of the
// 19 and within 7% of it on the others.  (profiles/launch_models.txt)
constexpr BlockModel TB2_MODEL[TB2_VARIANTS] = {{2, 0.295, 0.452, 2.7, 3.45}, {1, 0.281, 0, 2.9, 3.28},
                                                {1, 0.622, 0, 1.2, 3.73}, {2, 0.133, 0.225, 3.8, 3.02}};

// ns per step of a wavefront of R = 1, 2, 4 nodes per lane: alone on its SIMD
// (the dependent chain of a node) and each of several (their instructions).
constexpr double TB1_CHAIN[3] = {64, 86, 140}, TB1_ISSUE[3] = {43, 68, 120};

template <class F>
Shape1 best_shape1(F &&ns)
{
    Shape1 best;
    for (int i = 0; i < 3; ++i)
        for (int R = 1 << i, K = 8; K <= 32 * R - 4; K += 4) {
            const double t = ns(i, R, K);
            if (t < best.ns) best = Shape1{R, K, t};
        }
    return best;
}

// One wavefront per workgroup, launches 2 us apart.  With more than about 700
// wavefronts some of the 1024 SIMDs hold two.  (Measured: 1000 to 8000 nodes
// 122 to 130 ns at 2 nodes and 56 steps, 20011 138 at 2 / 48, 10^5 185 at
// 4 / 56, 10^6 692 at 4 / 28; the one-node-per-thread kernel takes 2.2 us.)
Shape1 tb1_shape(const Shape &s)
{
    return best_shape1([&](int i, int R, int K) {
        const double waves = (double)tb1_blocks(s, R, K);
        const double per = waves <= 700 ? 1.0 : ceil(waves / 1024.0 + (waves < 1024 ? 1.0 : 0.0));
        return 2000.0 / K + std::max(TB1_CHAIN[i], per * TB1_ISSUE[i]);
    });
}

// All in one workgroup of up to R1_WAVES wavefronts on four SIMDs, an exchange
// 320 ns (256 nodes: 101 ns per step at 1 node and 16 steps; 1500: 250).
Shape1 resident1_shape(const Shape &s)
{
    return best_shape1([&](int i, int R, int K) {
        const int64_t waves = tb1_blocks(s, R, K);
        if (waves > R1_WAVES) return 1e300;
        return 320.0 / K + std::max(TB1_CHAIN[i] + 10.0, (double)((waves + 3) / 4) * TB1_ISSUE[i]);
    });
}

bool tblock_applies(const ace_solver *s)
{
    if (s->p.d == 1) return tb1_supported(s->shape);
    return (s->p.d == 3 && tblock_supported(s->shape)) || (s->p.d == 2 && tblock2d_supported(s->shape));
}

int effective_kernel(const ace_solver *s)
{
    int k = s->kernel;
    if (k == ACE_KERNEL_AUTO) k = s->tuned_kernel;
    if (k == ACE_KERNEL_AUTO) k = s->rule_kernel;
    if (k == ACE_KERNEL_RESIDENT && s->p.total > RESIDENT_MAX) k = ACE_KERNEL_DIRECT;
    if (k == ACE_KERNEL_TBLOCK && !tblock_applies(s)) k = ACE_KERNEL_DIRECT;
    if (k == ACE_KERNEL_MARCH && !march_supported(s->shape)) k = ACE_KERNEL_DIRECT;
    return k;
}

// Steps one launch of `kernel` advances (in a long enough run).
// The register-resident 2D kernel is chosen and applies to the field.
bool use_tb2(const ace_solver *s) { return s->p.d == 2 && s->tb2 >= 0 && tb2_supported(s->shape); }

int steps_per_launch_of(const ace_solver *s, int kernel)
{
    if (kernel != ACE_KERNEL_TBLOCK) return 1;
    if (s->p.d == 1) return s->tb1.K;
    if (s->p.d == 3) return (s->tb3 >= 0 && tb3_supported(s->shape)) ? TB3_TABLE[s->tb3].depth : 2;
    return use_tb2(s) ? std::min(s->depth2, tb2_max_depth(s->tb2)) : s->depth2;
}

// Whether run_monitored at this interval is better with the whole field in one
// workgroup.  1D: a monitor costs it about 1.2 us, the launches of their own
// 3.  2D: a step takes 0.18 us and 0.235 ns per node (0.52 us at 40 x 40, 1.03
// at 64 x 64, 1.69 at 80 x 80), a monitor 1.5 us.
bool monitor_resident(const ace_solver *s, int64_t every)
{
    const double n = (double)s->p.total, steps = (double)every;
    if (n > RESIDENT_MAX) return false;
    if (s->p.d == 1) return s->res1.ns < 1e300 && 1200.0 + steps * s->res1.ns < 3000.0 + steps * s->tb1.ns;
    if (s->p.d != 2 || !use_tb2(s)) return false;
    const int K = std::min(s->depth2, tb2_max_depth(s->tb2)), rest = (int)(every % K);
    const BlockModel &m = TB2_MODEL[s->tb2];
    const double blocked = (double)(every / K) * m.us(tb2_blocks(s->tb2, s->shape, K), K) +
                           (rest ? m.us(tb2_blocks(s->tb2, s->shape, rest), rest) : 0.0);
    return 1.5 + steps * (0.18 + 2.35e-4 * n) < blocked;
}

bool on_tb2(const ace_solver *s, int K) { return use_tb2(s) && tb2_fits(s->tb2, s->shape, K); }

// One launch of the handle's 2D blocked kernel (K steps; level_stride > 0:
// every level written, as in launch_step_tblock2d): on its register regions,
// or on the LDS ones (of half the threads) where those are too many.
hipError_t launch_blocked2d(const ace_solver *s, const double *in, double *out, double *parts,
                            int64_t *nparts, int K, int64_t level_stride, hipStream_t st)
{
    if (on_tb2(s, K)) return launch_step_tb2(s->tb2, s->shape, s->coef, in, out, parts, nparts, K, level_stride, st);
    return launch_step_tblock2d(s->shape, s->coef, in, out, parts, nparts, K, level_stride, st);
}

int64_t blocked2d_blocks(const ace_solver *s, int K)
{
    return on_tb2(s, K) ? tb2_blocks(s->tb2, s->shape, K) : tblock2d_blocks(s->shape, K);
}

// The plane chunk of the handle's variant, unless it was set or tuned.
void follow_chunk(ace_solver *s)
{
    if (s->p.d != 3 || s->zchunk_fixed) return;
    std::vector<int> zcs;
    if (s->tb3 >= 0 && tb3_supported(s->shape)) zcs = tb3_chunks(s->tb3, s->shape, s->coef.fex);
    s->zchunk = zcs.empty() ? 32 : zcs[0];
}

// The rule's kernel and launch shape for a new handle.
// (Called again when the scheme changes: then only the tails, if the launch
// shape was set or tuned since.)
void plan_launch(ace_solver *s)
{
    const Shape &f = s->shape;
    if (!s->plan_fixed) s->rule_kernel = s->p.total <= RESIDENT_MAX ? ACE_KERNEL_RESIDENT : ACE_KERNEL_DIRECT;
    double best = 1e300;
    if (f.d == 2 && tb2_supported(f) && !s->plan_fixed) {
        for (int v = 0; v < TB2_VARIANTS; ++v)
            for (int K = 2; K <= std::min(tb2_max_depth(v), tblock2d_max_depth()); ++K) {
                const double us = TB2_MODEL[v].us(tb2_blocks(v, f, K), K) / K;
                if (tb2_max_depth(v) < tblock2d_max_depth() || us >= best) continue;  // (any depth stays settable)
                if (!tb2_fits(v, f, K)) continue;
                best = us;
                s->tb2 = v;
                s->depth2 = K;
            }
    }
    if (f.d == 1 && tb1_supported(f)) {
        s->tb1 = tb1_shape(f);
        if (f.M2 <= R1_MAX) s->res1 = resident1_shape(f);
        if (!s->plan_fixed)
            s->rule_kernel = s->res1.ns <= s->tb1.ns ? ACE_KERNEL_RESIDENT : ACE_KERNEL_TBLOCK;
    }
    // (2D: the LDS-resident kernel takes 0.52 us per step at 40 x 40 and 1.03
    // at 64 x 64, the blocked one 0.65 at both)
    if (f.d == 2 && s->p.total > 2048 && !s->plan_fixed &&
        (s->tb2 >= 0 || tblock2d_blocks(f, s->depth2) <= max_blocks(TBLOCK2D_THREADS)))
        s->rule_kernel = ACE_KERNEL_TBLOCK;
    if (f.d == 3 && tb3_supported(f)) {
        double of_depth[5] = {1e300, 1e300, 1e300, 1e300, 1e300};
        for (int v = 0; v < TB3_VARIANTS; ++v) {
            const std::vector<int> zcs = tb3_chunks(v, f, s->coef.fex);
            if (zcs.empty()) continue;
            const int zc = zcs[0], K = TB3_TABLE[v].depth;
            const double us = tb3_us(v, f, zc, s->coef.fex);
            if (us < of_depth[K]) {
                of_depth[K] = us;
                s->tail[K].v = v;
                s->tail[K].zchunk = zc;
            }
            if (us >= best || s->plan_fixed) continue;
            best = us;
            s->tb3 = v;
            if (!s->zchunk_fixed) s->zchunk = zc;
        }
    }
    if (s->plan_fixed) return;
    if (f.d == 3 && s->rule_kernel == ACE_KERNEL_DIRECT &&
        (s->tb3 < 0 || !col3d_supported(f) || kColumnUs + kColumnUsPerNode * (double)s->p.total > best))
        s->rule_kernel = ACE_KERNEL_TBLOCK;  // (without a region of k_tb3 the two-step kernel)
}

// The k_tb3 variant for a launch of `kernel` with `remaining` steps to go (-1:
// none): the handle's, or for a shorter rest of the run the fastest of that
// depth at its own plane chunk.
int tb3_for(const ace_solver *s, int kernel, int64_t remaining, int *zc)
{
    if (kernel != ACE_KERNEL_TBLOCK || s->p.d != 3 || s->tb3 < 0 || !tb3_supported(s->shape)) return -1;
    *zc = s->zchunk;
    if (remaining >= TB3_TABLE[s->tb3].depth) return s->tb3;
    *zc = s->tail[remaining].zchunk;
    return s->tail[remaining].v;
}

// One launch from in to out advancing 1 step, or up to steps_per_launch_of()
// with the temporal-blocking kernels; the monitor partials of in go to parts
// (if not null), their count to *nparts.  Returns the number of steps taken
// (or a negative error).
// Partial triples a monitored launch of `kernel` writes (the launch that
// launch_steps makes for `remaining` steps).
int64_t partials_for(const ace_solver *s, int kernel, int64_t remaining)
{
    if (kernel == ACE_KERNEL_TBLOCK && s->p.d == 1)
        return tb1_blocks(s->shape, s->tb1.R, (int)std::min<int64_t>(s->tb1.K, remaining));
    if (kernel == ACE_KERNEL_TBLOCK && s->p.d == 2)
        return blocked2d_blocks(s, (int)std::min<int64_t>(steps_per_launch_of(s, kernel), remaining));
    int zc = 0;
    const int v = tb3_for(s, kernel, remaining, &zc);
    if (v >= 0) return tb3_partials_needed(v, s->shape, zc);
    if (kernel == ACE_KERNEL_TBLOCK && remaining >= 2) return tblock_partials_needed(s->shape, s->zchunk);
    if (kernel == ACE_KERNEL_TBLOCK) kernel = one_step_kernel(s->shape);
    if (kernel == ACE_KERNEL_MARCH) return march_partials_needed(s->shape);
    return direct_partials_needed(s->shape);
}

int launch_between(const ace_solver *s, int kernel, const double *in, double *out, int64_t remaining, double *parts,
                   int64_t *nparts)
{
    hipError_t e;
    int taken = 1, zc = 0;
    const int v3 = tb3_for(s, kernel, remaining, &zc);
    if (kernel == ACE_KERNEL_TBLOCK && s->p.d == 1) {
        taken = (int)std::min<int64_t>(s->tb1.K, remaining);
        e = launch_step_tb1(s->shape, s->coef, in, out, parts, nparts, s->tb1.R, taken, s->stream);
    } else if (kernel == ACE_KERNEL_TBLOCK && s->p.d == 2) {
        taken = (int)std::min<int64_t>(steps_per_launch_of(s, kernel), remaining);
        e = launch_blocked2d(s, in, out, parts, nparts, taken, 0, s->stream);
    } else if (v3 >= 0) {
        e = launch_step_tb3(v3, s->shape, s->coef, in, out, parts, nparts, zc, s->stream);
        taken = TB3_TABLE[v3].depth;
    } else if (kernel == ACE_KERNEL_TBLOCK && remaining >= 2) {
        e = launch_step_tblock2(s->shape, s->coef, in, out, parts, nparts, s->zchunk, s->stream);
        taken = 2;
    } else if (kernel == ACE_KERNEL_MARCH ||
               (kernel == ACE_KERNEL_TBLOCK && one_step_kernel(s->shape) == ACE_KERNEL_MARCH)) {
        e = launch_step_march(s->shape, s->coef, in, out, parts, nparts, s->stream);
    } else {
        e = launch_step_direct(s->shape, s->coef, in, out, parts, nparts, s->stream);
    }
    ACE_HIP(e);
    return taken;
}

// The steps launch_between takes.
int64_t steps_of_launch(const ace_solver *s, int kernel, int64_t remaining)
{
    int zc = 0;
    const int v3 = tb3_for(s, kernel, remaining, &zc);
    if (v3 >= 0) return TB3_TABLE[v3].depth;
    if (kernel == ACE_KERNEL_TBLOCK && s->p.d == 3) return remaining >= 2 ? 2 : 1;
    return std::min<int64_t>(steps_per_launch_of(s, kernel), remaining);
}

// One launch from buf[cur] into buf[cur^1]; if want_mon, the monitor partials
// of the input field are left in s->partials, their count in *nparts.
int launch_steps(ace_solver *s, int kernel, int64_t remaining, bool want_mon, int64_t *nparts)
{
    if (want_mon && 3 * partials_for(s, kernel, remaining) > s->partials_cap) return ACE_E_STATE;
    const int taken = launch_between(s, kernel, s->buf[s->cur], s->buf[s->cur ^ 1], remaining,
                                     want_mon ? s->partials : nullptr, nparts);
    if (taken < 0) return taken;
    s->cur ^= 1;
    s->steps += taken;
    return taken;
}


// The whole run of `nsteps` in one workgroup (total <= RESIDENT_MAX).
hipError_t run_resident(const ace_solver *s, int64_t nsteps, int64_t every)
{
    double *f = s->buf[s->cur], *mon = every > 0 ? s->mon : nullptr;
    if (s->res1.ns < 1e300)
        return launch_resident1(s->shape, s->coef, f, nsteps, every, mon, s->res1.R, s->res1.K, s->stream);
    return launch_resident(s->shape, s->coef, f, nsteps, every, mon, s->stream);
}

void drop_graphs(ace_solver *s)
{
    // a replay may still run on the handle's stream
    if (!s->graphs.empty()) (void)hipStreamSynchronize(s->stream);
    for (auto &g : s->graphs) {
        (void)hipGraphExecDestroy(g.e);
        (void)hipGraphDestroy(g.g);
    }
    s->graphs.clear();
}

// Graph of s->graph_launches launches (an even count, so the field returns to
// the same buffer) of `kernel` starting from buf[cur]; captured once on a
// private stream and replayed on the handle's stream.  Kernel nodes only.
int graph_for(ace_solver *s, int kernel, hipGraphExec_t *out)
{
    for (auto &g : s->graphs)
        if (g.kernel == kernel && g.zchunk == s->zchunk && g.depth2 == s->depth2 && g.tb3 == s->tb3 &&
            g.tb2 == s->tb2 && g.cur == s->cur &&
            g.b0 == s->buf[0] && g.b1 == s->buf[1]) {
            *out = g.e;
            return ACE_OK;
        }
    if (!s->capture) ACE_HIP(hipStreamCreateWithFlags(&s->capture, hipStreamNonBlocking));
    const hipStream_t user = s->stream;
    const int cur0 = s->cur;
    const int64_t steps0 = s->steps;
    s->stream = s->capture;
    ACE_HIP(hipStreamBeginCapture(s->capture, hipStreamCaptureModeThreadLocal));
    int rc = ACE_OK;
    const int per = steps_per_launch_of(s, kernel);
    for (int64_t i = 0; i < s->graph_launches && rc >= 0; ++i) {
        const int t = launch_steps(s, kernel, per, false, nullptr);
        if (t < 0) rc = t;
    }
    hipGraph_t g = nullptr;
    hipError_t ce = hipStreamEndCapture(s->capture, &g);
    s->stream = user;
    s->cur = cur0;
    s->steps = steps0;
    if (rc < 0) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    ACE_HIP(ce);
    hipGraphExec_t e = nullptr;
    hipError_t ie = hipGraphInstantiate(&e, g, nullptr, nullptr, 0);
    if (ie != hipSuccess) {
        (void)hipGraphDestroy(g);
        return hip_status(ie);
    }
    s->graphs.push_back({kernel, s->zchunk, s->depth2, s->tb3, s->tb2, cur0, s->buf[0], s->buf[1], g, e});
    if (log_enabled())
        fprintf(stderr,
                "[ace] graph: %lld launches of kernel %d, %d step(s) each (plane chunk %d, 2D depth %d, "
                "3D variant %d)\n",
                (long long)s->graph_launches, kernel, per, s->zchunk, s->depth2, s->tb3);
    *out = e;
    return ACE_OK;
}

// Graph replays from buf[cur] for the first of nsteps steps, as long as two
// more graphs' steps are left; the steps taken go to *done.
int replay(ace_solver *s, int kernel, int64_t nsteps, int64_t *done)
{
    *done = 0;
    if (s->graph_launches < 2) return ACE_OK;
    const int64_t chunk = s->graph_launches * steps_per_launch_of(s, kernel);
    while (nsteps - *done >= 2 * chunk) {
        hipGraphExec_t e = nullptr;
        ACE_TRY(graph_for(s, kernel, &e));
        ACE_HIP(hipGraphLaunch(e, s->stream));
        s->steps += chunk;  // even launch count: s->cur is unchanged
        *done += chunk;
    }
    return ACE_OK;
}

int advance(ace_solver *s, int64_t nsteps)
{
    if (nsteps <= 0) return ACE_OK;
    const int k = effective_kernel(s);
    if (k == ACE_KERNEL_RESIDENT) {
        ACE_HIP(run_resident(s, nsteps, 0));
        s->steps += nsteps;
        return ACE_OK;
    }
    int64_t i = 0;
    ACE_TRY(replay(s, k, nsteps, &i));
    while (i < nsteps) {
        const int t = launch_steps(s, k, nsteps - i, false, nullptr);
        if (t < 0) return t;
        i += t;
    }
    return ACE_OK;
}

int alloc_fields(ace_solver *s)
{
    for (int i = 0; i < 2; ++i) {
        hipError_t e = hipMalloc((void **)&s->own[i], (size_t)s->p.total * sizeof(double));
        if (e != hipSuccess) return hip_status(e);
        s->buf[i] = s->own[i];
    }
    // one partial triple per workgroup of any monitored launch
    int64_t need2 = 3 * std::max<int64_t>(
        std::max<int64_t>(monitor_partials_needed(s->shape), direct_partials_needed(s->shape)), 1);
    if (tb1_supported(s->shape)) {
        const Shape1 t = tb1_shape(s->shape);
        need2 = std::max<int64_t>(need2, 3 * tb1_blocks(s->shape, t.R, t.K));
    }
    if (march_supported(s->shape)) need2 = std::max<int64_t>(need2, 3 * march_partials_needed(s->shape));
    if (tblock_supported(s->shape))
        need2 = std::max<int64_t>(need2, 3 * tblock_partials_needed(s->shape, TBLOCK_MIN_ZCHUNK));
    if (tb3_supported(s->shape))
        for (int v = 0; v < TB3_VARIANTS; ++v)
            need2 = std::max<int64_t>(need2, 3 * std::max<int64_t>(tb3_partials_needed(v, s->shape, 0),
                                                                 tb3_partials_needed(v, s->shape, TBLOCK_MIN_ZCHUNK)));
    if (tblock2d_supported(s->shape)) {
        need2 = std::max<int64_t>(need2, 3 * tblock2d_blocks(s->shape, tblock2d_max_depth()));
        if (tb2_supported(s->shape))
            for (int v = 0; v < TB2_VARIANTS; ++v)
                need2 = std::max<int64_t>(need2, 3 * tb2_blocks(v, s->shape, tb2_max_depth(v)));
    }
    ACE_TRY(grow(&s->partials, &s->partials_cap, need2));
    ACE_HIP(hipHostMalloc((void **)&s->pinned, 64 * sizeof(double), hipHostMallocDefault));
    return ACE_OK;
}

// Monitor triple of the current field into out[0..2] (device or
// pinned host memory; stream-ordered).
int monitor_now(ace_solver *s, double *out)
{
    int64_t np = 0;
    if (3 * monitor_partials_needed(s->shape) > s->partials_cap) return ACE_E_STATE;
    ACE_HIP(launch_monitor(s->shape, s->buf[s->cur], s->partials, &np, s->stream));
    ACE_HIP(launch_reduce(s->partials, np, out, s->stream));
    return ACE_OK;
}

// Monitor triple of the current field on the host: the reduction writes the
// handle's pinned memory.
int read_monitor(ace_solver *s, double *host3)
{
    ACE_TRY(monitor_now(s, s->pinned));
    ACE_HIP(hipStreamSynchronize(s->stream));
    memcpy(host3, s->pinned, 3 * sizeof(double));
    return ACE_OK;
}

// Region rows and depth of the reverse sweep with the least modelled time for
// a segment; false where no launch can hold the regions of both its kinds.
bool adj2_shape(const ace_solver *s, int *rows, int *K)
{
    const int64_t every = s->ck_every;
    double best = 1e300;
    for (int v = 0; v < 2; ++v)
        for (int d = 2; d <= std::min<int64_t>(12, std::max<int64_t>(every, 2)); ++d) {
            const int64_t launches = (std::min(every, s->ck_steps) + d - 1) / d;
            const int64_t blocks = 2 * adj2_tiles(s->shape, v ? 64 : 32, d);
            const double us = (double)launches * TB2_MODEL[v ? 2 : 1].us(blocks, d);
            if (us >= best || blocks > max_blocks(ADJ2_THREADS)) continue;
            best = us;
            *rows = v ? 64 : 32;
            *K = d;
        }
    return best < 1e300;
}

// Reverse sweep with the recompute of each segment in the launches of the one
// after it (ace_adj2.hip).  Leaves lambda^0 in lam[*lc], dL/dkappa in gsum.
int backward_regions(ace_solver *s, int rows, int K, double *const lam[2], int *lc)
{
    const int64_t total = s->p.total, every = s->ck_every, nsteps = s->ck_steps;
    const int n_tiles = (int)adj2_tiles(s->shape, rows, K);
    auto seg = [&](int64_t j) { return s->seg + (j & 1) * (every + 1) * total; };  // phi^{j every + 1} ..
    bool first = true;
    for (int64_t j = s->ck_count; j >= 0; --j) {
        // segment j backwards (j < ck_count) while segment j - 1 is recomputed
        const int64_t n = j < s->ck_count ? std::min<int64_t>(every, nsteps - j * every) : 0;
        const int64_t nf = j > 0 ? std::min<int64_t>(every, nsteps - (j - 1) * every) : 0;
        int64_t back = n, fwd = 0;  // steps of the segment left; states recomputed
        while (back > 0 || fwd < nf) {
            Adj2Args a = {};
            a.K = K;
            a.stride = total;
            a.Sr = (int)std::min<int64_t>(K, back);
            a.Sf = (int)std::min<int64_t>(K, nf - fwd);
            if (a.Sr > 0) {
                const int64_t m = back - a.Sr;  // the launch ends at state m of the segment
                a.n_rev = n_tiles;
                a.mu_in = lam[*lc];
                a.mu_out = lam[*lc ^ 1];
                a.phi_first = m == 0 ? s->ckpt + j * total : seg(j) + (m - 1) * total;
                a.phi_rest = seg(j) + m * total;
                a.phi_end = first ? seg(j) + (back - 1) * total : nullptr;
                a.last = j == 0 && m == 0;
                a.gpart = s->gpart;
                a.accumulate = !first;
            }
            if (a.Sf > 0) {
                a.f_in = fwd == 0 ? s->ckpt + (j - 1) * total : seg(j - 1) + (fwd - 1) * total;
                a.f_out = seg(j - 1) + fwd * total;
            }
            ACE_HIP(launch_adj2(rows, s->shape, s->coef, a, s->stream));
            if (a.Sr > 0) {
                *lc ^= 1;
                first = false;
            }
            back -= a.Sr;
            fwd += a.Sf;
        }
    }
    ACE_HIP(launch_sum(s->gpart, n_tiles, s->gsum, 0, s->stream));
    return ACE_OK;
}

// Reverse sweep step by step; the recompute of segment j-1 runs on a second
// stream while segment j is swept backwards on the handle's, on alternating
// segment buffers: events order each buffer's recompute after the previous
// sweep that used it, and each sweep after its recompute.
int backward_steps(ace_solver *s, int k, double *const lam[2], int *lc)
{
    const int64_t total = s->p.total, every = s->ck_every, nsteps = s->ck_steps;
    const size_t bytes = (size_t)total * sizeof(double);
    const int64_t npart = adjoint_partials_needed(s->shape);
    const bool columns = adjoint_col_supported(s->shape);  // mu form, one sum for the sweep
    const bool blocked2d = (k == ACE_KERNEL_TBLOCK && s->p.d == 2);
    if (k == ACE_KERNEL_TBLOCK && !blocked2d) k = one_step_kernel(s->shape);
    if (!s->aux) ACE_HIP(hipStreamCreateWithFlags(&s->aux, hipStreamNonBlocking));
    if (!s->ev_start) {
        ACE_HIP(hipEventCreateWithFlags(&s->ev_start, hipEventDisableTiming));
        for (int b = 0; b < 2; ++b) {
            ACE_HIP(hipEventCreateWithFlags(&s->ev_rec[b], hipEventDisableTiming));
            ACE_HIP(hipEventCreateWithFlags(&s->ev_rev[b], hipEventDisableTiming));
        }
    }
    if (!columns) ACE_HIP(hipMemsetAsync(s->gsum, 0, sizeof(double), s->stream));
    ACE_HIP(hipEventRecord(s->ev_start, s->stream));  // checkpoints are complete
    ACE_HIP(hipStreamWaitEvent(s->aux, s->ev_start, 0));
    bool first = true;
    for (int64_t j = s->ck_count - 1; j >= 0; --j) {
        const int b = (int)(j & 1);
        double *seg = s->seg + b * (every + 1) * total;
        const int64_t a = j * every;
        const int64_t n = std::min<int64_t>(every, nsteps - a);
        // --- recompute segment j on the second stream ---
        ACE_HIP(hipStreamWaitEvent(s->aux, s->ev_rev[b], 0));
        ACE_HIP(hipMemcpyAsync(seg, s->ckpt + j * total, bytes, hipMemcpyDeviceToDevice, s->aux));
        if (blocked2d) {
            const int per = steps_per_launch_of(s, ACE_KERNEL_TBLOCK);
            for (int64_t i = 0; i < n;) {  // each launch writes its K intermediate states
                const int K = (int)std::min<int64_t>(per, n - i);
                ACE_HIP(launch_blocked2d(s, seg + i * total, seg + (i + 1) * total, nullptr, nullptr, K, total,
                                         s->aux));
                i += K;
            }
        } else {
            for (int64_t i = 0; i < n; ++i) {
                const double *in = seg + i * total;
                double *out = seg + (i + 1) * total;
                hipError_t e = (k == ACE_KERNEL_MARCH)
                                   ? launch_step_march(s->shape, s->coef, in, out, nullptr, nullptr, s->aux)
                                   : launch_step_direct(s->shape, s->coef, in, out, nullptr, nullptr, s->aux);
                ACE_HIP(e);
            }
        }
        ACE_HIP(hipEventRecord(s->ev_rec[b], s->aux));
        // --- reverse sweep of segment j on the handle's stream ---
        ACE_HIP(hipStreamWaitEvent(s->stream, s->ev_rec[b], 0));
        int64_t parts = 0;  // partial sums of dL/dkappa written for this segment
        if (blocked2d) {
            // (deeper launches leave the 32-row regions of the reverse sweep small tiles)
            const int rev = std::min(s->depth2, 8);
            for (int64_t i = n; i > 0;) {  // K transposed steps per launch
                const int K = (int)std::min<int64_t>(rev, i);
                ACE_HIP(launch_adjoint_tblock2d(s->shape, s->coef, lam[*lc], seg + (i - K) * total, total,
                                                lam[*lc ^ 1], s->gpart + parts, K, s->stream));
                parts += tblock2d_blocks(s->shape, K);
                *lc ^= 1;
                i -= K;
            }
        } else {
            for (int64_t i = n - 1; i >= 0; --i) {
                if (columns) {
                    ACE_HIP(launch_adjoint_col(s->shape, s->coef, lam[*lc], seg + i * total,
                                               first ? seg + (i + 1) * total : nullptr, lam[*lc ^ 1], s->gpart,
                                               j == 0 && i == 0, !first, s->stream));
                    first = false;
                } else {
                    ACE_HIP(launch_adjoint_step(s->shape, s->coef, lam[*lc], seg + i * total,
                                                seg + (i + 1) * total, lam[*lc ^ 1], s->gpart + parts, nullptr,
                                                s->stream));
                    parts += npart;
                }
                *lc ^= 1;
            }
        }
        if (parts > 0) ACE_HIP(launch_sum(s->gpart, parts, s->gsum, 1, s->stream));
        ACE_HIP(hipEventRecord(s->ev_rev[b], s->stream));
    }
    if (columns) ACE_HIP(launch_sum(s->gpart, adjoint_col_blocks(s->shape), s->gsum, 0, s->stream));
    return ACE_OK;
}

// Autotuner cache: one JSON object per line and tuned problem shape,
//   {"d": 2, "bc": 0, "M": [1024, 1024, 1], "kernel": 4, "zchunk": 32,
//    "depth2": 5, "tb3": -1, "tb2": 0, "ms_per_step": 0.003389}
// appended by ace_autotune (kTuneFormat) and read back with the same format;
// the last matching line wins, other lines are skipped.
constexpr const char *kTuneFormat =
    "{\"d\": %d, \"bc\": %d, \"M\": [%lld, %lld, %lld], \"kernel\": %d, \"zchunk\": %d, "
    "\"depth2\": %d, \"tb3\": %d, \"tb2\": %d, \"ms_per_step\": %lf}";

void load_tuning(ace_solver *s)
{
    const char *path = getenv("ACE_AUTOTUNE_CACHE");
    if (!path) return;
    FILE *f = fopen(path, "r");
    if (!f) return;
    char line[512];
    while (fgets(line, sizeof line, f)) {
        int d, bc, k, zc, k2, v3, v2;
        long long m0, m1, m2;
        double ms;
        if (sscanf(line, kTuneFormat, &d, &bc, &m0, &m1, &m2, &k, &zc, &k2, &v3, &v2, &ms) != 11) continue;
        if (d == s->p.d && bc == s->p.bc && m0 == s->p.M[0] && m1 == s->p.M[1] && m2 == s->p.M[2] &&
            k >= ACE_KERNEL_DIRECT && k <= ACE_KERNEL_TBLOCK &&
            (zc == 0 || zc >= TBLOCK_MIN_ZCHUNK) && k2 >= 1 && k2 <= tblock2d_max_depth() && v3 >= -1 &&
            v3 < TB3_VARIANTS && v2 >= -1 && v2 < TB2_VARIANTS) {
            s->tuned_kernel = k;
            s->zchunk = zc;
            s->zchunk_fixed = 1;
            s->plan_fixed = 1;
            s->depth2 = k2;
            s->tb3 = v3;
            s->tb2 = v2;
        }
    }
    fclose(f);
}

}  // namespace

extern "C" {

const char *ace_version(void) { return "ace-mi355x 0.1 (gfx950, fp64)"; }

const char *ace_strerror(int st)
{
    switch (st) {
    case ACE_OK: return "ok";
    case ACE_E_ARG: return "invalid argument";
    case ACE_E_SIZE: return "too few cells for the boundary condition";
    case ACE_E_ANISO: return "grid spacing differs between axes";
    case ACE_E_DT: return "time step outside (0, 2): the cubic has no unique real root";
    case ACE_E_HIP: return "HIP runtime error";
    case ACE_E_NOMEM: return "out of memory";
    case ACE_E_NONFINITE: return "non-finite value in the field";
    case ACE_E_STATE: return "call not valid in the current state";
    case ACE_W_CONDITIONS: return "warning: dt > 1 - 2 d kappa (maximum-principle condition fails)";
    case ACE_W_PHI0_GT1: return "warning: |phi0| > 1 somewhere";
    case ACE_W_MAXPRINCIPLE: return "warning: max-norm exceeded 1 under the step condition";
    case ACE_W_ENERGY_UP: return "warning: energy increased under the step condition";
    default: return "unknown status";
    }
}

int ace_create(int d, const int64_t *N, const double *L, const double *R, double eps, double dt,
               int bc, ace_solver **out)
{
    if (!out) return ACE_E_ARG;
    *out = nullptr;
    Problem p;
    const int rc = derive(d, N, L, R, eps, dt, bc, p);
    if (rc < 0) return rc;
    ace_solver *s = new (std::nothrow) ace_solver();
    if (!s) return ACE_E_NOMEM;
    s->p = p;
    s->shape = shape_of(p);
    s->coef = coef_of(p);
    (void)hipGetDevice(&s->device);
    scratch_setup(s->device);
    const int arc = alloc_fields(s);
    if (arc < 0) {
        ace_destroy(s);
        return arc;
    }
    plan_launch(s);
    load_tuning(s);
    hipError_t e = hipMalloc((void **)&s->gsum, 4 * sizeof(double));
    if (e != hipSuccess) {
        ace_destroy(s);
        return hip_status(e);
    }
    if (log_enabled())
        fprintf(stderr, "[ace] create d=%d bc=%d M=%lldx%lldx%lld dx=%.6g kappa=%.6g h=%.6g Newton steps %d%s%s\n",
                p.d, p.bc, (long long)p.M[0], (long long)p.M[1], (long long)p.M[2], p.dx, p.kappa, p.h, p.nit,
                p.start2 ? " (second-order start)" : "", p.cond_ok ? "" : ", outside Theorem 2's conditions");
    *out = s;
    return rc;
}

int ace_destroy(ace_solver *s)
{
    if (!s) return ACE_E_ARG;
    drop_graphs(s);
    if (s->capture) (void)hipStreamDestroy(s->capture);
    if (s->aux) (void)hipStreamDestroy(s->aux);
    hipEvent_t evs[] = {s->ev_start, s->ev_rec[0], s->ev_rec[1], s->ev_rev[0], s->ev_rev[1]};
    for (hipEvent_t e : evs)
        if (e) (void)hipEventDestroy(e);
    for (int i = 0; i < 2; ++i)
        if (s->own[i]) (void)hipFree(s->own[i]);
    double *devs[] = {s->partials, s->mon, s->monparts, s->ckpt, s->seg, s->lam, s->gpart, s->gsum};
    for (double *p : devs)
        if (p) (void)hipFree(p);
    if (s->pinned) (void)hipHostFree(s->pinned);
    delete s;
    return ACE_OK;
}

int ace_shape(const ace_solver *s, int64_t M[3], int64_t *total)
{
    if (!s) return ACE_E_ARG;
    if (M)
        for (int j = 0; j < 3; ++j) M[j] = s->p.M[j];
    if (total) *total = s->p.total;
    return ACE_OK;
}

int ace_node_coords(const ace_solver *s, int axis, double *x)
{
    if (!s || !x || axis < 0 || axis >= s->p.d) return ACE_E_ARG;
    const double L = s->p.L[axis], dx = s->p.dx;
    for (int64_t i = 0; i < s->p.M[axis]; ++i) {
        // Sec. 2: x_i = dx (i - 1/2) for HN, dx i for HD (i = 1..N-1) and P
        if (s->p.bc == ACE_BC_HN) x[i] = L + ((double)i - 0.5) * dx;
        else if (s->p.bc == ACE_BC_HD) x[i] = L + (double)(i + 1) * dx;
        else x[i] = L + (double)i * dx;
    }
    return ACE_OK;
}

int ace_params(const ace_solver *s, ace_params_t *q)
{
    if (!s || !q) return ACE_E_ARG;
    memset(q, 0, sizeof(*q));
    const Problem &p = s->p;
    q->d = p.d;
    q->bc = p.bc;
    for (int j = 0; j < 3; ++j) {
        q->N[j] = p.N[j];
        q->M[j] = p.M[j];
    }
    q->total = p.total;
    q->dx = p.dx;
    q->dt = p.dt;
    q->eps = p.eps;
    q->kappa = p.kappa;
    q->h = p.h;
    q->dt_bound = p.dx * p.dx / (p.dx * p.dx + 2.0 * p.d * p.eps * p.eps);
    // Sec. 4: omega_1 = 1/3, 1/5, 1/6 for d = 1, 2, 3; s = omega_1 / kappa
    q->omega1 = (p.d == 1) ? 1.0 / 3.0 : (p.d == 2 ? 0.2 : 1.0 / 6.0);
    q->s = q->omega1 / p.kappa;
    q->conditions_ok = p.cond_ok;
    q->newton_iters = p.nit;
    q->scheme = p.scheme;
    return ACE_OK;
}

int ace_set_stream(ace_solver *s, void *st)
{
    if (!s) return ACE_E_ARG;
    if ((hipStream_t)st != s->stream) {
        leave_stream(s->stream, (hipStream_t)st);
        drop_graphs(s);  // a replay on the old stream may still use a captured graph
    }
    s->stream = (hipStream_t)st;
    return ACE_OK;
}

int ace_bind_fields(ace_solver *s, double *a, double *b)
{
    if (!s) return ACE_E_ARG;
    if ((a == nullptr) != (b == nullptr) || (a && a == b)) return ACE_E_ARG;
    if (a) {
        s->buf[0] = a;
        s->buf[1] = b;
    } else {
        s->buf[0] = s->own[0];
        s->buf[1] = s->own[1];
    }
    s->cur = 0;
    s->steps = 0;
    s->field_version++;
    drop_graphs(s);
    return ACE_OK;
}

int ace_set_graph_launches(ace_solver *s, int64_t launches)
{
    if (!s || launches < 0) return ACE_E_ARG;
    s->graph_launches = launches + (launches & 1);  // even: the buffer parity returns
    drop_graphs(s);
    return ACE_OK;
}

int ace_set_eps(ace_solver *s, double eps)
{
    if (!s) return ACE_E_ARG;
    if (!(eps > 0.0) || !isfinite(eps)) return ACE_E_ARG;
    s->ck_count = 0;  // checkpoints of the old eps are no longer valid
    if (eps != s->p.eps) {
        // only kappa and the conditions depend on eps
        s->p.eps = eps;
        s->p.kappa = eps * eps * s->p.dt / (s->p.dx * s->p.dx);
        set_conditions(s->p);
        s->coef = coef_of(s->p);
        drop_graphs(s);  // captured launches carry the old coefficients
    }
    return s->p.cond_ok ? ACE_OK : ACE_W_CONDITIONS;
}

int ace_set_scheme(ace_solver *s, int scheme)
{
    if (!s || (scheme != ACE_SCHEME_RLB_MIE && scheme != ACE_SCHEME_FEX)) return ACE_E_ARG;
    s->p.scheme = scheme;
    set_conditions(s->p);
    s->coef = coef_of(s->p);
    plan_launch(s);
    s->ck_count = 0;
    drop_graphs(s);
    return s->p.cond_ok ? ACE_OK : ACE_W_CONDITIONS;
}

int ace_set_kernel(ace_solver *s, int kernel, int depth)
{
    if (!s || kernel < ACE_KERNEL_AUTO || kernel > ACE_KERNEL_TBLOCK || depth < 0) return ACE_E_ARG;
    if (kernel == ACE_KERNEL_TBLOCK && depth != 0) {
        if (s->p.d == 3 && (depth < 2 || depth > 4)) return ACE_E_ARG;
        if (s->p.d == 2 && depth > tblock2d_max_depth()) return ACE_E_ARG;
        if (s->p.d == 2) s->depth2 = depth;
        if (s->p.d == 3) s->tb3 = (depth == 2) ? -1 : (depth == 3 ? TB3_DEFAULT_DEPTH3 : TB3_DEFAULT_DEPTH4);
        s->plan_fixed = 1;
        follow_chunk(s);
    }
    s->kernel = kernel;
    s->depth = depth;
    return ACE_OK;
}

int ace_set_region3d(ace_solver *s, int depth, int rows, int rows_per_thread)
{
    if (!s || s->p.d != 3) return ACE_E_ARG;
    if (depth == 2 && rows == 0 && rows_per_thread == 0) {
        s->tb3 = -1;
        s->plan_fixed = 1;
        follow_chunk(s);
        return ACE_OK;
    }
    const int v = tb3_find(depth, rows, rows_per_thread);
    if (v < 0) return ACE_E_ARG;
    s->tb3 = v;
    s->plan_fixed = 1;
    follow_chunk(s);
    return ACE_OK;
}

int ace_get_region3d(const ace_solver *s, int *depth, int *rows, int *rows_per_thread)
{
    if (!s || !depth || !rows || !rows_per_thread || s->p.d != 3) return ACE_E_ARG;
    if (s->tb3 < 0) {
        *depth = 2;
        *rows = 0;
        *rows_per_thread = 0;
    } else {
        *depth = TB3_TABLE[s->tb3].depth;
        *rows = TB3_TABLE[s->tb3].rows;
        *rows_per_thread = TB3_TABLE[s->tb3].rpt;
    }
    return ACE_OK;
}

int ace_set_region2d(ace_solver *s, int rows, int rows_per_thread)
{
    if (!s || s->p.d != 2) return ACE_E_ARG;
    if (rows == 0 && rows_per_thread == 0) {
        s->tb2 = -1;
        s->plan_fixed = 1;
        return ACE_OK;
    }
    const int v = tb2_find(rows, rows_per_thread);
    if (v < 0) return ACE_E_ARG;
    s->tb2 = v;
    s->plan_fixed = 1;
    return ACE_OK;
}

int ace_get_region2d(const ace_solver *s, int *rows, int *rows_per_thread)
{
    if (!s || !rows || !rows_per_thread || s->p.d != 2) return ACE_E_ARG;
    *rows = s->tb2 >= 0 ? TB2_TABLE[s->tb2].rows : 0;
    *rows_per_thread = s->tb2 >= 0 ? TB2_TABLE[s->tb2].rpt : 0;
    return ACE_OK;
}

int ace_set_plane_chunk(ace_solver *s, int planes)
{
    if (!s || s->p.d != 3 || (planes != 0 && (planes < TBLOCK_MIN_ZCHUNK || planes > 4096)))
        return ACE_E_ARG;
    s->zchunk = planes;
    s->zchunk_fixed = 1;
    return ACE_OK;
}

int ace_get_plane_chunk(const ace_solver *s, int *planes)
{
    if (!s || !planes) return ACE_E_ARG;
    *planes = s->zchunk;
    return ACE_OK;
}

int ace_get_kernel(const ace_solver *s, int *kernel, int *steps_per_launch)
{
    if (!s || !kernel) return ACE_E_ARG;
    const int k = effective_kernel(s);
    *kernel = k;
    if (steps_per_launch) *steps_per_launch = steps_per_launch_of(s, k);
    return ACE_OK;
}

int ace_set_phi0(ace_solver *s, const double *phi0, int where)
{
    if (!s || !phi0 || (where != ACE_HOST && where != ACE_DEVICE)) return ACE_E_ARG;
    int warn = ACE_OK;
    const size_t bytes = (size_t)s->p.total * sizeof(double);
    if (where == ACE_HOST) {
        for (int64_t i = 0; i < s->p.total; ++i) {
            if (!isfinite(phi0[i])) return ACE_E_NONFINITE;
            if (fabs(phi0[i]) > 1.0) warn = ACE_W_PHI0_GT1;
        }
        ACE_HIP(hipMemcpyAsync(s->buf[0], phi0, bytes, hipMemcpyHostToDevice, s->stream));
        ACE_HIP(hipStreamSynchronize(s->stream));
    } else {
        ACE_HIP(hipMemcpyAsync(s->buf[0], phi0, bytes, hipMemcpyDeviceToDevice, s->stream));
    }
    s->cur = 0;
    s->steps = 0;
    s->field_version++;
    return warn;
}

int ace_step(ace_solver *s, int64_t nsteps)
{
    if (!s || nsteps < 0) return ACE_E_ARG;
    ACE_TRY(advance(s, nsteps));
    s->field_version++;
    return ACE_OK;
}

int ace_run_monitored(ace_solver *s, int64_t nsteps, int64_t every, double *E, double *maxn)
{
    if (!s || nsteps < 0 || every < 1 || !E || !maxn) return ACE_E_ARG;
    const int64_t nmon = nsteps / every + 1;
    ACE_TRY(grow(&s->mon, &s->mon_cap, 3 * nmon));
    int k = effective_kernel(s);
    if (s->kernel == ACE_KERNEL_AUTO && s->tuned_kernel == ACE_KERNEL_AUTO && monitor_resident(s, every))
        k = ACE_KERNEL_RESIDENT;
    if (k == ACE_KERNEL_RESIDENT) {
        ACE_HIP(run_resident(s, nsteps, every));
        s->steps += nsteps;
    } else {
        // The partials of up to `batch` monitors are kept and reduced together
        // (one launch instead of one per monitor, as long as they take less
        // than 32 MB), all of a run's equal intervals alike.  np0: the most
        // partials of an interval's launch; a persistent grid writes fewer.
        const int64_t np0 = partials_for(s, k, std::min<int64_t>(every, std::max<int64_t>(nsteps, 1)));
        const int64_t batch = std::max<int64_t>(1, std::min<int64_t>(nmon, ((int64_t)1 << 22) / (3 * np0)));
        // (without that memory each monitor is reduced by itself, as are those
        // of which only one fits)
        const bool many = batch > 1 && grow(&s->monparts, &s->monparts_cap, batch * 3 * np0) >= 0;
        if (batch > 1 && !many) (void)hipGetLastError();
        int64_t j = 0, kept = 0, npk = 0;  // monitors done, of them not reduced yet, and their partials
        auto flush = [&]() -> int {
            if (kept > 0)
                ACE_HIP(launch_reduce_many(s->monparts, npk, 3 * np0, kept, s->mon + 3 * (j - kept), s->stream));
            kept = 0;
            return ACE_OK;
        };
        for (int64_t st = 0; st <= nsteps; st += every) {
            if (st == nsteps) {
                ACE_TRY(flush());
                ACE_TRY(monitor_now(s, s->mon + 3 * j));
            } else {
                const int64_t seg = std::min<int64_t>(every, nsteps - st);
                const int64_t want = partials_for(s, k, seg);
                const bool keep = many && want == np0;
                if (!keep || kept == batch) ACE_TRY(flush());
                int64_t np = 0;
                double *parts = keep ? s->monparts + 3 * np0 * kept : s->partials;
                if (!keep && 3 * want > s->partials_cap) return ACE_E_STATE;
                int64_t done = launch_between(s, k, s->buf[s->cur], s->buf[s->cur ^ 1], seg, parts, &np);
                if (done < 0) return (int)done;
                s->cur ^= 1;
                s->steps += done;
                if (kept > 0 && np != npk) ACE_TRY(flush());  // (their slots are read before this one's is reused)
                if (keep && parts == s->monparts + 3 * np0 * kept) {
                    ++kept;
                    npk = np;
                } else {
                    ACE_HIP(launch_reduce(parts, np, s->mon + 3 * j, s->stream));
                }
                while (done < seg) {
                    const int t = launch_steps(s, k, seg - done, false, nullptr);
                    if (t < 0) return t;
                    done += t;
                }
            }
            ++j;
            if (st == nsteps) break;
        }
        if (kept > 0) ACE_TRY(flush());
    }
    s->field_version++;
    std::vector<double> trip((size_t)(3 * nmon));
    ACE_HIP(hipMemcpyAsync(trip.data(), s->mon, trip.size() * sizeof(double), hipMemcpyDeviceToHost,
                           s->stream));
    ACE_HIP(hipStreamSynchronize(s->stream));
    for (int64_t j = 0; j < nmon; ++j) {
        E[j] = energy_from(s->p, &trip[3 * j]);
        maxn[j] = trip[3 * j + 2];
    }
    return ace_monitor_status(nmon, E, maxn, s->p.cond_ok, &s->warn_mask);
}

int ace_get_warnings(const ace_solver *s, int *mask)
{
    if (!s || !mask) return ACE_E_ARG;
    *mask = s->warn_mask;
    return ACE_OK;
}

int ace_monitor_status(int64_t n, const double *E, const double *maxn, int conditions_ok, int *mask)
{
    if (mask) *mask = 0;
    if (n < 1 || !E || !maxn) return ACE_E_ARG;
    int bits = 0;
    for (int64_t j = 0; j < n; ++j) {
        if (!isfinite(maxn[j]) || !isfinite(E[j])) return ACE_E_NONFINITE;
        if (!conditions_ok) continue;
        // Theorem 2: |phi| <= 1 is kept; Theorem 3: the energy does not rise
        if (maxn[j] > 1.0 + 4.0 * 0x1p-53) bits |= ACE_WARN_BIT(ACE_W_MAXPRINCIPLE);
        if (j > 0 && E[j] > E[j - 1] + 1e-14 * fabs(E[j - 1])) bits |= ACE_WARN_BIT(ACE_W_ENERGY_UP);
    }
    if (mask) *mask = bits;
    if (bits & ACE_WARN_BIT(ACE_W_MAXPRINCIPLE)) return ACE_W_MAXPRINCIPLE;
    if (bits & ACE_WARN_BIT(ACE_W_ENERGY_UP)) return ACE_W_ENERGY_UP;
    return ACE_OK;
}

int ace_energy(ace_solver *s, double *E)
{
    if (!s || !E) return ACE_E_ARG;
    double t[3];
    ACE_TRY(read_monitor(s, t));
    *E = energy_from(s->p, t);
    return isfinite(*E) ? ACE_OK : ACE_E_NONFINITE;
}

int ace_maxnorm(ace_solver *s, double *m)
{
    if (!s || !m) return ACE_E_ARG;
    double t[3];
    ACE_TRY(read_monitor(s, t));
    *m = t[2];
    return isfinite(*m) ? ACE_OK : ACE_E_NONFINITE;
}

int ace_phase_volume(ace_solver *s, double *V)
{
    if (!s || !V) return ACE_E_ARG;
    ACE_TRY(grow(&s->partials, &s->partials_cap, phase_partials_needed()));
    ACE_HIP(launch_phase_volume(s->buf[s->cur], s->p.total, s->partials, s->pinned, s->stream));
    ACE_HIP(hipStreamSynchronize(s->stream));
    *V = pow(s->p.dx, s->p.d) * s->pinned[0];
    return isfinite(*V) ? ACE_OK : ACE_E_NONFINITE;
}

int ace_monitor_noalloc(ace_solver *s, const double *phi, double *out)
{
    if (!s || !out) return ACE_E_ARG;
    double *scr = scratch_of(s->device);
    if (!scr) return ACE_E_STATE;
    const int64_t np = monitor_partials_needed(s->shape);
    if (np < 1 || np > kNoAllocParts) return ACE_E_SIZE;
    const double *f = phi ? phi : s->buf[s->cur];
    int64_t n2 = 0;
    ACE_HIP(launch_monitor(s->shape, f, scr + kTripSlot, &n2, s->stream));
    ACE_HIP(launch_reduce(scr + kTripSlot, n2, scr, s->stream));
    double dxd, cg;
    energy_coefs(s->p, &dxd, &cg);
    ACE_HIP(launch_monitor_finish(scr, dxd, cg, out, s->stream));
    return ACE_OK;
}

int ace_equivalent_radius(ace_solver *s, double *R)
{
    if (!s || !R) return ACE_E_ARG;
    double V = 0.0;
    ACE_TRY(ace_phase_volume(s, &V));
    // Sec. 4.2.2: the circle (V = pi R^2) and the sphere (V = 4/3 pi R^3);
    // in 1D the phase is an interval of length 2R
    if (s->p.d == 1) *R = 0.5 * V;
    else if (s->p.d == 2) *R = sqrt(V / M_PI);
    else *R = cbrt(3.0 * V / (4.0 * M_PI));
    return isfinite(*R) ? ACE_OK : ACE_E_NONFINITE;
}

int ace_get_phi(ace_solver *s, double *out, int where)
{
    if (!s || !out || (where != ACE_HOST && where != ACE_DEVICE)) return ACE_E_ARG;
    const size_t bytes = (size_t)s->p.total * sizeof(double);
    ACE_HIP(hipMemcpyAsync(out, s->buf[s->cur], bytes,
                           where == ACE_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice,
                           s->stream));
    if (where == ACE_HOST) ACE_HIP(hipStreamSynchronize(s->stream));
    return ACE_OK;
}

int64_t ace_step_count(const ace_solver *s) { return s ? s->steps : -1; }

const double *ace_field_ptr(const ace_solver *s) { return s ? s->buf[s->cur] : nullptr; }

// Shortest timed trial of the autotuner, and the most steps a lengthened
// trial may take.
constexpr double kMinTrialMs = 2.0;
constexpr int64_t kMaxTrialSteps = 1 << 20;

int ace_autotune(ace_solver *s, int64_t trial_steps, char *json, size_t cap)
{
    if (!s || trial_steps < 1) return ACE_E_ARG;
    struct Cand {
        int kernel, zchunk, depth2, tb3, tb2;
    };
    std::vector<Cand> cands;
    const int z0c = s->zchunk, k0 = s->depth2, v30 = s->tb3, v20 = s->tb2;
    cands.push_back({ACE_KERNEL_DIRECT, z0c, k0, v30, v20});
    if (s->p.total <= RESIDENT_MAX) cands.push_back({ACE_KERNEL_RESIDENT, z0c, k0, v30, v20});
    if (s->p.d == 1 && tb1_supported(s->shape)) cands.push_back({ACE_KERNEL_TBLOCK, z0c, k0, v30, v20});
    if (march_supported(s->shape)) cands.push_back({ACE_KERNEL_MARCH, z0c, k0, v30, v20});
    if (s->p.d == 3 && tblock_supported(s->shape))
        for (int zc : {0, 32})  // 0: persistent grid
            if (zc <= std::max<int64_t>(s->shape.M0, 16)) cands.push_back({ACE_KERNEL_TBLOCK, zc, k0, -1, v20});
    // the configurable 3D kernel: every depth and region shape, as a
    // persistent grid and at the three plane chunks with the least modelled
    // time (the least one where the field is so small that a launch is one
    // round of workgroups at any of them).  The deep 48-row region is timed
    // where it has workgroups for half of the CUs (on smaller fields it never
    // came near the others).
    if (s->p.d == 3 && tb3_supported(s->shape))
        for (int v = 0; v < TB3_VARIANTS; ++v) {
            if (v >= TB3_NAMED && tb3_partials_needed(v, s->shape, 16) < 128) continue;
            std::vector<int> zcs = tb3_chunks(v, s->shape, s->coef.fex);
            zcs.resize(std::min<size_t>(zcs.size(), s->p.total < 100000 ? 1 : 3));
            zcs.push_back(0);
            for (int zc : zcs) cands.push_back({ACE_KERNEL_TBLOCK, zc, k0, v, v20});
        }
    if (s->p.d == 2 && tblock2d_supported(s->shape)) {
        for (int k2 : {1, 2, 3, 4, 5, 6, 8, 10, 12})
            if (k2 <= tblock2d_max_depth()) cands.push_back({ACE_KERNEL_TBLOCK, z0c, k2, v30, -1});
        // the register-resident 2D kernel: every region shape and depth
        for (int v = 0; v < (tb2_supported(s->shape) ? TB2_VARIANTS : 0); ++v)
            for (int k2 : {2, 3, 4, 5, 6, 8, 10, 12})
                if (k2 <= tb2_max_depth(v)) cands.push_back({ACE_KERNEL_TBLOCK, z0c, k2, v30, v});
    }
    const int64_t total = s->p.total;
    double *save = nullptr;
    ACE_HIP(hipMalloc((void **)&save, sizeof(double) * total));
    const int cur0 = s->cur;
    const int64_t steps0 = s->steps;
    const int kernel0 = s->kernel, zchunk0 = s->zchunk, depth20 = s->depth2, tb30 = s->tb3, tb20 = s->tb2;
    int rc = hip_status(hipMemcpyAsync(save, s->buf[cur0], sizeof(double) * total,
                                       hipMemcpyDeviceToDevice, s->stream));
    auto restore = [&]() {
        s->cur = cur0;
        return hip_status(hipMemcpyAsync(s->buf[cur0], save, sizeof(double) * total,
                                         hipMemcpyDeviceToDevice, s->stream));
    };
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (rc >= 0) rc = hip_status(hipEventCreate(&e0));
    if (rc >= 0) rc = hip_status(hipEventCreate(&e1));
    // restores the field, then times `n` steps on the handle's stream
    auto time_run = [&](int64_t n, float *out) -> int {
        int r;
        if ((r = restore()) < 0) return r;
        if ((r = hip_status(hipEventRecord(e0, s->stream))) < 0) return r;
        if ((r = advance(s, n)) < 0) return r;
        if ((r = hip_status(hipEventRecord(e1, s->stream))) < 0) return r;
        if ((r = hip_status(hipEventSynchronize(e1))) < 0) return r;
        return hip_status(hipEventElapsedTime(out, e0, e1));
    };
    std::string rec = "{\"kind\": \"solver\", \"trial_steps\": " + std::to_string(trial_steps) +
                      ", \"candidates\": [";
    double best_ms = 1e300;
    Cand best = cands[0];
    bool first = true;
    for (const Cand &c : cands) {
        if (rc < 0) break;
        s->kernel = c.kernel;
        s->zchunk = c.zchunk;
        s->depth2 = c.depth2;
        s->tb3 = c.tb3;
        s->tb2 = c.tb2;
        // Each length is run once untimed (code object load, graph capture)
        // and then timed.  A trial shorter than kMinTrialMs is lengthened to
        // about that, so small fields are timed in the steady state of a long
        // run (graph replay) rather than on a few directly issued launches.
        int64_t steps = trial_steps;
        float ms = 0.f;
        if ((rc = time_run(steps, &ms)) < 0) break;
        if ((rc = time_run(steps, &ms)) < 0) break;
        if (ms < kMinTrialMs && steps < kMaxTrialSteps) {
            const double scale = kMinTrialMs / std::max<double>(ms, 1e-3);
            steps = std::min<int64_t>(kMaxTrialSteps, (int64_t)ceil((double)steps * scale));
            if ((rc = time_run(steps, &ms)) < 0) break;
            if ((rc = time_run(steps, &ms)) < 0) break;
        }
        const double per = ms / (double)steps;
        char buf[320];
        const int d3 = c.tb3 >= 0 ? TB3_TABLE[c.tb3].depth : 2;
        const int r3 = c.tb3 >= 0 ? TB3_TABLE[c.tb3].rows : 0, t3 = c.tb3 >= 0 ? TB3_TABLE[c.tb3].rpt : 0;
        const int r2 = c.tb2 >= 0 ? TB2_TABLE[c.tb2].rows : 0, t2 = c.tb2 >= 0 ? TB2_TABLE[c.tb2].rpt : 0;
        snprintf(buf, sizeof buf,
                 "%s{\"kernel\": %d, \"zchunk\": %d, \"depth2\": %d, \"tb3\": %d, \"depth3\": %d, "
                 "\"rows\": %d, \"rows_per_thread\": %d, \"tb2\": %d, \"rows2\": %d, "
                 "\"rows_per_thread2\": %d, \"steps\": %lld, \"ms_per_step\": %.6f}",
                 first ? "" : ", ", c.kernel, c.zchunk, c.depth2, c.tb3, d3, r3, t3, c.tb2, r2, t2, (long long)steps,
                 per);
        rec += buf;
        first = false;
        if (per < best_ms) {
            best_ms = per;
            best = c;
        }
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    s->kernel = kernel0;
    s->zchunk = zchunk0;
    s->depth2 = depth20;
    s->tb3 = tb30;
    s->tb2 = tb20;
    if (rc >= 0) rc = restore();
    if (rc >= 0) rc = hip_status(hipStreamSynchronize(s->stream));
    (void)hipFree(save);
    s->steps = steps0;
    if (rc < 0) return rc;
    s->tuned_kernel = best.kernel;
    s->zchunk = best.zchunk;
    s->zchunk_fixed = 1;
    s->plan_fixed = 1;
    s->depth2 = best.depth2;
    s->tb3 = best.tb3;
    s->tb2 = best.tb2;
    drop_graphs(s);
    char buf[320];
    {
        const int d3 = best.tb3 >= 0 ? TB3_TABLE[best.tb3].depth : 2;
        const int r3 = best.tb3 >= 0 ? TB3_TABLE[best.tb3].rows : 0;
        const int t3 = best.tb3 >= 0 ? TB3_TABLE[best.tb3].rpt : 0;
        const int r2 = best.tb2 >= 0 ? TB2_TABLE[best.tb2].rows : 0;
        const int t2 = best.tb2 >= 0 ? TB2_TABLE[best.tb2].rpt : 0;
        snprintf(buf, sizeof buf,
                 "], \"choice\": {\"kernel\": %d, \"zchunk\": %d, \"depth2\": %d, \"tb3\": %d, "
                 "\"depth3\": %d, \"rows\": %d, \"rows_per_thread\": %d, \"tb2\": %d, \"rows2\": %d, "
                 "\"rows_per_thread2\": %d, \"ms_per_step\": %.6f}}",
                 best.kernel, best.zchunk, best.depth2, best.tb3, d3, r3, t3, best.tb2, r2, t2, best_ms);
    }
    rec += buf;
    if (json && cap > 0) snprintf(json, cap, "%s", rec.c_str());
    if (log_enabled())
        fprintf(stderr,
                "[ace] autotune d=%d bc=%d M=%lldx%lldx%lld: kernel %d, plane chunk %d, 2D depth %d, "
                "3D variant %d, 2D variant %d, %.6f ms/step\n",
                s->p.d, s->p.bc, (long long)s->p.M[0], (long long)s->p.M[1], (long long)s->p.M[2], best.kernel,
                best.zchunk, best.depth2, best.tb3, best.tb2, best_ms);
    const char *path = getenv("ACE_AUTOTUNE_CACHE");
    if (path) {
        FILE *f = fopen(path, "a");
        if (f) {
            // the same fields as kTuneFormat, ms written with a fixed precision
            fprintf(f,
                    "{\"d\": %d, \"bc\": %d, \"M\": [%lld, %lld, %lld], \"kernel\": %d, \"zchunk\": %d, "
                    "\"depth2\": %d, \"tb3\": %d, \"tb2\": %d, \"ms_per_step\": %.6f}\n",
                    s->p.d, s->p.bc, (long long)s->p.M[0], (long long)s->p.M[1], (long long)s->p.M[2],
                    best.kernel, best.zchunk, best.depth2, best.tb3, best.tb2, best_ms);
            fclose(f);
        }
    }
    return ACE_OK;
}

// ---------------------------------------------------------------------------
// reverse mode
// ---------------------------------------------------------------------------

int ace_forward_ckpt(ace_solver *s, const double *phi0, int where, int64_t nsteps, int64_t every)
{
    if (!s || !phi0 || nsteps < 0 || every < 1) return ACE_E_ARG;
    if (s->p.scheme != ACE_SCHEME_RLB_MIE) return ACE_E_STATE;
    const int rc = ace_set_phi0(s, phi0, where);
    if (rc < 0) return rc;
    const int64_t total = s->p.total;
    const int64_t nck = nsteps == 0 ? 1 : (nsteps + every - 1) / every;
    ACE_TRY(grow(&s->ckpt, &s->ckpt_cap, nck * total));
    // size the reverse sweep's buffers now so ace_backward allocates nothing
    ACE_TRY(grow(&s->seg, &s->seg_cap, 2 * (every + 1) * total));
    ACE_TRY(grow(&s->lam, &s->lam_cap, 2 * total));
    int64_t parts = adjoint_partials_needed(s->shape) * every;
    if (adjoint_col_supported(s->shape)) parts = std::max(parts, adjoint_col_blocks(s->shape));
    if (tblock2d_supported(s->shape)) {
        parts = std::max<int64_t>(parts, tblock2d_blocks(s->shape, tblock2d_max_depth()) * every);
        if (tb2_supported(s->shape)) parts = std::max(parts, adj2_tiles(s->shape, 32, 12));
    }
    ACE_TRY(grow(&s->gpart, &s->gpart_cap, parts));
    const size_t bytes = (size_t)total * sizeof(double);
    const int k = effective_kernel(s);
    const double *in = s->buf[s->cur];
    int64_t in_ckpt = 0;  // steps the field at `in` is ahead of buf[cur], whose count is s->steps
    ACE_HIP(hipMemcpyAsync(s->ckpt, in, bytes, hipMemcpyDeviceToDevice, s->stream));
    for (int64_t j = 0; j < nck; ++j) {
        int64_t left = std::min<int64_t>(every, nsteps - j * every);
        if (k == ACE_KERNEL_RESIDENT) {  // in place
            ACE_TRY(advance(s, left));
            if (j + 1 < nck)
                ACE_HIP(hipMemcpyAsync(s->ckpt + (j + 1) * total, s->buf[s->cur], bytes, hipMemcpyDeviceToDevice,
                                       s->stream));
            continue;
        }
        // a segment's last launch writes the next checkpoint, which the next
        // segment's first launch reads; graphs replay what lies between
        while (left > 0) {
            if (in == s->buf[s->cur]) {
                int64_t done = 0;
                ACE_TRY(replay(s, k, left, &done));
                left -= done;
            }
            double *out = s->buf[s->cur ^ 1];
            const int64_t t = steps_of_launch(s, k, left);
            if (t == left && j + 1 < nck) out = s->ckpt + (j + 1) * total;
            const int taken = launch_between(s, k, in, out, left, nullptr, nullptr);
            if (taken < 0) return taken;
            if (taken != t) return ACE_E_STATE;
            left -= taken;
            in_ckpt += taken;
            if (out == s->buf[s->cur ^ 1]) {
                s->cur ^= 1;
                s->steps += in_ckpt;
                in_ckpt = 0;
            }
            in = out;
        }
    }
    s->field_version++;
    s->ck_every = every;
    s->ck_steps = nsteps;
    s->ck_count = nck;
    s->ck_field_version = s->field_version;
    s->ck_generation++;
    return rc;
}

int64_t ace_ckpt_generation(const ace_solver *s) { return s ? s->ck_generation : -1; }

int ace_backward(ace_solver *s, const double *lambdaT, double *dphi0, double *deps2, int where)
{
    if (!s || !lambdaT || !dphi0 || !deps2 || (where != ACE_HOST && where != ACE_DEVICE))
        return ACE_E_ARG;
    if (s->ck_count <= 0 || s->ck_field_version != s->field_version) return ACE_E_STATE;
    const int64_t total = s->p.total, every = s->ck_every, nsteps = s->ck_steps;
    const size_t bytes = (size_t)total * sizeof(double);
    if (s->seg_cap < 2 * (every + 1) * total || s->lam_cap < 2 * total) return ACE_E_STATE;
    double *lam[2] = {s->lam, s->lam + total};
    int lc = 0, rows = 0, K = 0;
    int k = effective_kernel(s);
    if (k == ACE_KERNEL_RESIDENT) k = ACE_KERNEL_DIRECT;
    ACE_HIP(hipMemcpyAsync(lam[0], lambdaT, bytes,
                           where == ACE_HOST ? hipMemcpyHostToDevice : hipMemcpyDeviceToDevice,
                           s->stream));
    if (nsteps == 0) {
        ACE_HIP(hipMemsetAsync(s->gsum, 0, sizeof(double), s->stream));
    } else if (k == ACE_KERNEL_TBLOCK && use_tb2(s) && adj2_shape(s, &rows, &K)) {
        ACE_TRY(backward_regions(s, rows, K, lam, &lc));
    } else {
        ACE_TRY(backward_steps(s, k, lam, &lc));
    }
    ACE_HIP(hipMemcpyAsync(dphi0, lam[lc], bytes,
                           where == ACE_HOST ? hipMemcpyDeviceToHost : hipMemcpyDeviceToDevice,
                           s->stream));
    ACE_HIP(hipMemcpyAsync(s->pinned, s->gsum, sizeof(double), hipMemcpyDeviceToHost, s->stream));
    ACE_HIP(hipStreamSynchronize(s->stream));
    // kappa = eps^2 dt / dx^2  =>  dL/d(eps^2) = (dt / dx^2) dL/dkappa
    *deps2 = s->pinned[0] * s->p.dt / (s->p.dx * s->p.dx);
    return ACE_OK;
}

int ace_adjoint(ace_solver *s, const double *phi0, int64_t nsteps, int64_t ckpt_every,
                const double *lambdaT, double *dphi0, double *deps2, int where)
{
    const int rc = ace_forward_ckpt(s, phi0, where, nsteps, ckpt_every);
    if (rc < 0) return rc;
    return ace_backward(s, lambdaT, dphi0, deps2, where);
}

}  // extern "C"
