/* Host-only stand-in for the HIP runtime calls that libnbody.so makes, so that
 * the host side of the C ABI can be followed without a GPU (test_host_calls.py):
 * "device" memory is host memory, copies and fills are done at once, kernels
 * are not run but written to a log, and a stream's wait returns stub_sync_rc. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } Dim;
#define API __attribute__((visibility("default")))

API int stub_sync_rc = 0;         /* what hipStreamSynchronize returns */
API int stub_mapped_rc = 0;       /* what hipHostGetDevicePointer returns for old blocks */
API int stub_mallocs = 0, stub_frees = 0;
API void *stub_block = 0;         /* the last hipHostMalloc */

enum { MAXF = 4096, MAXL = 256 };
static struct { const void *f; const char *name; } fn[MAXF];
static int n_fn;
/* log of launches: kernel name (mangled), grid, and the partial-sum argument
 * (the fourth) of an evaluation kernel */
API int stub_launches = 0;
static struct { const char *name; uint32_t gx, gy; void *part; } lg[MAXL];
API const char *stub_name(int k) { return lg[k].name; }
API uint32_t stub_gx(int k) { return lg[k].gx; }
API uint32_t stub_gy(int k) { return lg[k].gy; }
API void *stub_part(int k) { return lg[k].part; }

API void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
API void __hipUnregisterFatBinary(void **m) { (void)m; }
API void __hipRegisterVar(void) {}
API void __hipRegisterFunction(void **m, const void *f, char *df, const char *name)
{
    (void)m; (void)df;
    if (n_fn < MAXF) {
        fn[n_fn].f = f;
        fn[n_fn++].name = name;
    }
}

static struct { Dim g, b; size_t sh; void *s; } cfg;
API int __hipPushCallConfiguration(Dim g, Dim b, size_t sh, void *s)
{
    cfg.g = g; cfg.b = b; cfg.sh = sh; cfg.s = s;
    return 0;
}
API int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *sh, void **s)
{
    *g = cfg.g; *b = cfg.b; *sh = cfg.sh; *s = cfg.s;
    return 0;
}
API int hipLaunchKernel(const void *f, Dim g, Dim b, void **args, size_t sh, void *s)
{
    const char *name = "?";
    (void)b; (void)sh; (void)s;
    for (int k = 0; k < n_fn; ++k)
        if (fn[k].f == f)
            name = fn[k].name;
    if (stub_launches < MAXL) {
        lg[stub_launches].name = name;
        lg[stub_launches].gx = g.x;
        lg[stub_launches].gy = g.y;
        lg[stub_launches].part = strstr(name, "12force_kernel") ? *(void **)args[3] : 0;
        ++stub_launches;
    }
    return 0;
}
API int hipLaunchCooperativeKernel(const void *f, Dim g, Dim b, void **a, unsigned sh, void *s)
{
    (void)f; (void)g; (void)b; (void)a; (void)sh; (void)s;
    return 1;
}

API int hipGetDevice(int *d) { *d = 0; return 0; }
API int hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 0; return 0; }
API int hipGetLastError(void) { return 0; }
API const char *hipGetErrorString(int e) { (void)e; return "stub"; }
API int hipGetSymbolAddress(void **p, const void *s)
{
    (void)s;
    *p = (void *)(uintptr_t)0x100000000;   /* never dereferenced: kernels do not run */
    return 0;
}
API int hipHostMalloc(void **p, size_t n, unsigned f)
{
    (void)f;
    ++stub_mallocs;
    stub_block = *p = calloc(1, n);
    return 0;
}
API int hipHostFree(void *p) { ++stub_frees; (void)p; return 0; }   /* kept: addresses stay distinct */
API int hipHostGetDevicePointer(void **d, void *h, unsigned f)
{
    (void)f;
    *d = h;
    return h == stub_block ? 0 : stub_mapped_rc;
}
API int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st)
{
    (void)k; (void)st;
    memmove(d, s, n);
    return 0;
}
API int hipMemsetAsync(void *d, int v, size_t n, void *st)
{
    (void)st;
    memset(d, v, n);
    return 0;
}
API int hipStreamSynchronize(void *s) { (void)s; return stub_sync_rc; }
API int hipStreamQuery(void *s) { (void)s; return 0; }
API int hipEventCreate(void **e) { *e = 0; return 0; }
API int hipEventDestroy(void *e) { (void)e; return 0; }
API int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
API int hipEventSynchronize(void *e) { (void)e; return 0; }
API int hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 0; return 0; }
API int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *v, const void *f, int b, size_t sh)
{
    (void)f; (void)b; (void)sh;
    *v = 0;
    return 0;
}
