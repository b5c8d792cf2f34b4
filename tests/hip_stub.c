/* A stand-in for the HIP runtime on hosts without a GPU: device memory is
 * reserved host memory, kernels do nothing, and every launch, graph replay,
 * synchronisation and wait is logged as one line of text.  Loaded with
 * RTLD_GLOBAL before the library, it is what the library's host code then
 * calls (tests/hip_stub.py). */
#define _GNU_SOURCE
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

typedef struct {
    uint32_t x, y, z;
} dim3_t;
enum { OK = 0, NOMEM = 2, BADCONFIG = 9, LAUNCHFAIL = 719 };

static char *g_log;
static size_t g_len, g_cap;
static int64_t g_launches_left = -1;               /* launches until one fails (-1: none does) */
static uint64_t g_refuse_from = UINT64_MAX;        /* smallest allocation that is refused */
static struct { const void *host; char *name; } g_fn[65536];
static int g_nfn;
static void *g_capturing[16];
static dim3_t g_grid, g_block;
static size_t g_shm;
static void *g_stream;

static void put(const char *line)
{
    const size_t n = strlen(line);
    if (g_len + n + 1 > g_cap) {
        g_cap = 2 * g_cap + n + 4096;
        g_log = realloc(g_log, g_cap);
    }
    memcpy(g_log + g_len, line, n + 1);
    g_len += n;
}
const char *stub_log(void) { return g_log ? g_log : ""; }
void stub_clear(void)
{
    g_len = 0;
    put("");
}
void stub_fail_launch(int64_t after) { g_launches_left = after; }
void stub_refuse_from(uint64_t bytes) { g_refuse_from = bytes; }
void stub_set_capturing(void *s, int on)
{
    for (int i = 0; i < 16; ++i)
        if (g_capturing[i] == (on ? NULL : s)) {
            g_capturing[i] = on ? s : NULL;
            return;
        }
}
static int capturing(void *s)
{
    for (int i = 0; i < 16; ++i)
        if (s && g_capturing[i] == s) return 1;
    return 0;
}

int hipMalloc(void **p, size_t n)
{
    *p = NULL;
    if (n >= g_refuse_from) return NOMEM;
    /* (the size is kept in front, for hipFree) */
    size_t *m = mmap(NULL, n + 4096, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return NOMEM;
    m[0] = n;
    *p = (char *)m + 4096;
    return OK;
}
int hipFree(void *p)
{
    if (p) munmap((char *)p - 4096, *(size_t *)((char *)p - 4096) + 4096);
    return OK;
}
int hipHostMalloc(void **p, size_t n, unsigned f) { return (*p = calloc(1, n)) ? OK : NOMEM; }
int hipHostFree(void *p) { free(p); return OK; }
int hipMemcpy(void *d, const void *s, size_t n, int k)
{
    if (n <= ((size_t)1 << 26)) memmove(d, s, n);
    return OK;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st)
{
    char line[96];
    snprintf(line, sizeof line, "copy %zu on %p\n", n, st);
    put(line);
    return hipMemcpy(d, s, n, k);
}
int hipMemcpy2DAsync(void *d, size_t dp, const void *s, size_t sp, size_t w, size_t h, int k, void *st) { return OK; }
int hipMemset(void *d, int v, size_t n) { return OK; }
int hipMemsetAsync(void *d, int v, size_t n, void *st) { return OK; }

int hipStreamCreateWithFlags(void **s, unsigned f) { return (*s = malloc(8)) ? OK : NOMEM; }
int hipStreamDestroy(void *s) { free(s); return OK; }
int hipStreamSynchronize(void *s)
{
    char line[64];
    snprintf(line, sizeof line, "%s %p\n", capturing(s) ? "broken-capture" : "sync", s);
    put(line);
    return capturing(s) ? 900 : OK;
}
int hipStreamIsCapturing(void *s, int *st) { *st = capturing(s); return OK; }
int hipStreamBeginCapture(void *s, int m) { stub_set_capturing(s, 1); return OK; }
int hipStreamEndCapture(void *s, void **g)
{
    stub_set_capturing(s, 0);
    *g = malloc(8);
    return OK;
}
int hipStreamWaitEvent(void *s, void *e, unsigned f) { return OK; }
int hipGraphInstantiate(void **e, void *g, void *n, char *b, size_t z) { *e = malloc(8); put("instantiate\n"); return OK; }
int hipGraphLaunch(void *e, void *s) { put("replay\n"); return OK; }
int hipGraphExecDestroy(void *e) { free(e); return OK; }
int hipGraphDestroy(void *g) { free(g); return OK; }
int hipEventCreate(void **e) { *e = malloc(8); return OK; }
int hipEventCreateWithFlags(void **e, unsigned f) { return hipEventCreate(e); }
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventRecord(void *e, void *s) { return OK; }
int hipEventSynchronize(void *e) { return OK; }
static float g_ms = 1.0f, g_ms_step;
void stub_elapsed(float first, float step) /* each time asked for: first, first + step, ... */
{
    g_ms = first;
    g_ms_step = step;
}
int hipEventElapsedTime(float *t, void *a, void *b)
{
    *t = g_ms;
    g_ms += g_ms_step;
    return OK;
}
int hipGetDevice(int *d) { *d = 0; return OK; }
int hipDeviceGetAttribute(int *v, int a, int d) { *v = 256; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *f, int b, size_t m) { *v = 1; return OK; }
static int g_last;
int hipGetLastError(void) { const int e = g_last; g_last = OK; return e; }
const char *hipGetErrorString(int e) { return "stub error"; }
int hipGetSymbolAddress(void **p, const void *s) { *p = NULL; return NOMEM; }

void **__hipRegisterFatBinary(const void *d) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) {}
void __hipRegisterVar(void **h, void *v, char *a, char *b, int e, size_t n, int c, int g) {}
void __hipRegisterFunction(void **h, const void *f, char *d, const char *name, unsigned t, void *a, void *b, void *c,
                           void *e, int *w)
{
    if (g_nfn == 65536) return;
    g_fn[g_nfn].host = f;
    g_fn[g_nfn++].name = strdup(name);
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t shm, void *st)
{
    g_grid = g;
    g_block = b;
    g_shm = shm;
    g_stream = st;
    return OK;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *shm, void **st)
{
    *g = g_grid;
    *b = g_block;
    *shm = g_shm;
    *st = g_stream;
    return OK;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t shm, void *st)
{
    const char *name = "?";
    char line[1024];
    for (int i = 0; i < g_nfn; ++i)
        if (g_fn[i].host == f) name = g_fn[i].name;
    g_last = OK;
    if ((uint64_t)g.x * b.x >> 32 || (uint64_t)g.y * b.y >> 32 || (uint64_t)g.z * b.z >> 32 || !g.x) g_last = BADCONFIG;
    if (g_launches_left == 0) g_last = LAUNCHFAIL;
    if (g_launches_left >= 0) --g_launches_left;
    snprintf(line, sizeof line, "%s %s grid %u %u %u block %u on %p args %p %p\n", g_last ? "refused" : "launch", name,
             g.x, g.y, g.z, b.x, st, *(void **)args[0], *(void **)args[1]);
    put(line);
    return g_last;
}
