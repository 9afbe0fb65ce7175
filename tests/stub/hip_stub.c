/* A HIP runtime of the calls the library makes, on host memory and with no
 * device, for CPU tests of its host code: launches are counted and do nothing;
 * hipMalloc fails where the test says.  As in the runtime, a failed call sets
 * the thread's last error, which stays until hipGetLastError takes it. */
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef int hipError_t;
typedef struct { uint32_t x, y, z; } dim3;
enum { ok = 0, invalid_value = 1, out_of_memory = 2 };

static hipError_t last;
static int mallocs, frees, launches;
static uint64_t bytes, sizes[64];
static uint64_t fail_mask; /* bit i: the i-th hipMalloc from now fails */
static dim3 grid_, block_;
static size_t shared_;
static void *stream_;
static char symbol_[256];

void stub_fail_mallocs(uint64_t mask) { mallocs = frees = launches = 0; bytes = 0; fail_mask = mask; }
int stub_mallocs(void) { return mallocs; }
uint64_t stub_bytes(void) { return bytes; } /* asked for in all */
uint64_t stub_size(int i) { return sizes[i]; } /* by the i-th hipMalloc */
int stub_frees(void) { return frees; }
int stub_launches(void) { return launches; }

static hipError_t set(hipError_t e) { if (e != ok) last = e; return e; }
hipError_t hipGetLastError(void) { hipError_t e = last; last = ok; return e; }
hipError_t hipPeekAtLastError(void) { return last; }
const char *hipGetErrorString(hipError_t e) { return e == ok ? "no error" : e == out_of_memory ? "out of memory" : "error"; }

hipError_t hipMalloc(void **p, size_t n)
{
    const int i = mallocs++;
    bytes += n;
    if (i < 64) sizes[i] = n;
    *p = i < 64 && (fail_mask >> i & 1) ? NULL : aligned_alloc(256, (n + 255) & ~(size_t)255);
    if (*p) return ok;
    ++frees; /* nothing to free */
    return set(out_of_memory);
}
hipError_t hipFree(void *p) { frees += p != NULL; free(p); return ok; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return ok; }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return ok; }

hipError_t hipGetDevice(int *d) { *d = 0; return ok; }
hipError_t hipDeviceGetAttribute(int *v, int attr, int d) { (void)attr; (void)d; *v = 8; return ok; }
hipError_t hipGetDevicePropertiesR0600(void *prop, int d) { (void)prop; (void)d; return set(invalid_value); }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l)
{
    (void)f; (void)b; (void)l;
    *n = 2;
    return ok;
}
hipError_t hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return ok; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = symbol_; return ok; }

hipError_t hipStreamCreate(void **s) { *s = symbol_; return ok; }
hipError_t hipStreamDestroy(void *s) { (void)s; return ok; }
hipError_t hipEventCreate(void **e) { *e = symbol_; return ok; }
hipError_t hipEventDestroy(void *e) { (void)e; return ok; }
hipError_t hipEventRecord(void *e, void *s) { (void)e; (void)s; return ok; }
hipError_t hipEventSynchronize(void *e) { (void)e; return ok; }
hipError_t hipEventElapsedTime(float *t, void *a, void *b) { (void)a; (void)b; *t = 1.f; return ok; }

hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t l, void *s)
{
    (void)f; (void)g; (void)b; (void)args; (void)l; (void)s;
    ++launches;
    return ok;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, void *s)
{
    grid_ = g;
    block_ = b;
    shared_ = l;
    stream_ = s;
    return ok;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, void **s)
{
    *g = grid_;
    *b = block_;
    *l = shared_;
    *s = stream_;
    return ok;
}
void **__hipRegisterFatBinary(const void *data) { static void *m; (void)data; return &m; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *h, char *d, const char *n, unsigned l, void *a, void *b, void *c,
                           void *e, int *w)
{
    (void)m; (void)h; (void)d; (void)n; (void)l; (void)a; (void)b; (void)c; (void)e; (void)w;
}
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t n, int c, int g)
{
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)n; (void)c; (void)g;
}
