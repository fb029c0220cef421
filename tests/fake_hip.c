/* A HIP runtime for tests of the library's host code without a GPU: device
 * memory is host memory, a copy is a memcpy, streams, events and graphs are
 * numbers, and a kernel launch only appends the kernel's name to a log.  After
 * fake_fail_after(n) the n+1st launch from then on fails (n < 0: none). */
#define _GNU_SOURCE
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef int err_t;
enum { kOk = 0, kFail = 719 };

enum { kMaxFn = 4096, kMaxLog = 1 << 20 };
static struct { const void *fn; const char *name; } g_fn[kMaxFn];
static int g_n_fn, g_fail_after = -1;
static char g_log[kMaxLog];
static size_t g_len;
static err_t g_last;
static dim3_t g_grid, g_block;
static size_t g_shmem;
static void *g_stream;
static uintptr_t g_handle = 16;

const char *fake_log(void) { return g_log; }
void fake_reset(void) { g_len = 0; g_log[0] = 0; }
void fake_fail_after(int n) { g_fail_after = n; }

void **__hipRegisterFatBinary(const void *data) { (void)data; static void *h; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **m, const void *host, char *dev, const char *name, unsigned limit, void *a, void *b,
                           void *c, void *d, int *w) {
    (void)m; (void)dev; (void)limit; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (g_n_fn < kMaxFn) { g_fn[g_n_fn].fn = host; g_fn[g_n_fn++].name = name; }
}
void __hipRegisterVar(void **m, void *var, char *host, char *dev, int ext, size_t size, int cst, int glob) {
    (void)m; (void)var; (void)host; (void)dev; (void)ext; (void)size; (void)cst; (void)glob;
}
err_t __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t sh, void *st) {
    g_grid = g; g_block = b; g_shmem = sh; g_stream = st;
    return kOk;
}
err_t __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *sh, void **st) {
    *g = g_grid; *b = g_block; *sh = g_shmem; *st = g_stream;
    return kOk;
}
err_t hipLaunchKernel(const void *fn, dim3_t g, dim3_t b, void **args, size_t sh, void *st) {
    (void)args; (void)sh; (void)st;
    if (g_fail_after == 0) return g_last = kFail;
    if (g_fail_after > 0) --g_fail_after;
    const char *name = "?";
    for (int k = 0; k < g_n_fn; ++k)
        if (g_fn[k].fn == fn) name = g_fn[k].name;
    if (g_len + strlen(name) + 64 < kMaxLog)
        g_len += (size_t)sprintf(g_log + g_len, "%s %u %u\n", name, g.x * g.y * g.z, b.x);
    return kOk;
}
err_t hipGetLastError(void) { err_t e = g_last; g_last = kOk; return e; }
const char *hipGetErrorString(err_t e) { return e ? "failed as asked" : "no error"; }

err_t hipMalloc(void **p, size_t n) { *p = aligned_alloc(256, (n + 255) / 256 * 256 + 256); return *p ? kOk : 2; }
err_t hipFree(void *p) { free(p); return kOk; }
err_t hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return kOk; }
err_t hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
    (void)kind; (void)st; memcpy(d, s, n);
    return kOk;
}
err_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)288 << 30; return kOk; }
err_t hipGetDevice(int *d) { *d = 0; return kOk; }
err_t hipGetDeviceCount(int *n) { *n = 1; return kOk; }
err_t hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 160 * 1024; return kOk; }
err_t hipGetSymbolAddress(void **p, const void *sym) {
    (void)sym;
    static void *mem;
    if (!mem) mem = aligned_alloc(256, (size_t)96 << 20);
    *p = mem;
    return mem ? kOk : 2;
}

static err_t handle(void **h) { *h = (void *)(g_handle += 16); return kOk; }
err_t hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; return handle(s); }
err_t hipStreamDestroy(void *s) { (void)s; return kOk; }
err_t hipStreamSynchronize(void *s) { (void)s; return kOk; }
err_t hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return kOk; }
err_t hipStreamBeginCapture(void *s, int mode) { (void)s; (void)mode; return kOk; }
err_t hipStreamEndCapture(void *s, void **g) { (void)s; return handle(g); }
err_t hipGraphInstantiate(void **x, void *g, void **n, char *b, size_t s) {
    (void)g; (void)n; (void)b; (void)s;
    return handle(x);
}
err_t hipGraphLaunch(void *x, void *s) { (void)x; (void)s; return kOk; }
err_t hipGraphDestroy(void *g) { (void)g; return kOk; }
err_t hipGraphExecDestroy(void *x) { (void)x; return kOk; }
err_t hipEventCreate(void **e) { return handle(e); }
err_t hipEventCreateWithFlags(void **e, unsigned f) { (void)f; return handle(e); }
err_t hipEventDestroy(void *e) { (void)e; return kOk; }
err_t hipEventRecord(void *e, void *s) { (void)e; (void)s; return kOk; }
err_t hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return kOk; }
