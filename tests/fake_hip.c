/* The HIP runtime calls that libpam_lattice.so makes, without a GPU: device
 * allocations are addresses that nothing reads, they and launches are recorded, and
 * the build's compaction publishes the outcome that the test sets, so that
 * the library's own launch sequence, grids and buffer handling run on the
 * CPU.  Loaded with RTLD_GLOBAL before the library, whose calls then resolve
 * here.  Like the runtime, a launch of 2^32 work items or more in one
 * dimension is refused. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
    uint32_t x, y, z;
} dim3;

enum { kOk = 0, kOutOfMemory = 2, kInvalidConfiguration = 9 };

static char g_log[1 << 20];
static size_t g_len;
static uint32_t g_count, g_flags, g_bucket;
static uint64_t g_fail_above = ~0ull;
static uint64_t g_next = 0x100000000000ull;
static int g_error;
static dim3 g_grid, g_block;

/* ---- for the test */
void fake_outcome(uint32_t count, uint32_t flags, uint32_t nbucket)
{
    g_count = count;
    g_flags = flags;
    g_bucket = nbucket;
}
void fake_fail_above(uint64_t bytes) { g_fail_above = bytes; }
const char *fake_log(void) { return g_log; }
void fake_clear(void)
{
    g_len = 0;
    g_log[0] = 0;
}

/* ---- the runtime */
int hipMalloc(void **p, size_t bytes)
{
    if (bytes > g_fail_above)
        return kOutOfMemory;
    g_len += (size_t)snprintf(g_log + g_len, sizeof g_log - g_len, "malloc %zu\n", bytes);
    *p = (void *)g_next;
    g_next += (bytes + 0xffff) & ~(uint64_t)0xffff;
    return kOk;
}
int hipFree(void *p)
{
    (void)p;
    return kOk;
}
int hipHostMalloc(void **p, size_t bytes, unsigned flags)
{
    (void)flags;
    *p = calloc(1, bytes);
    return *p ? kOk : kOutOfMemory;
}
int hipHostFree(void *p)
{
    free(p);
    return kOk;
}
int hipGetDevice(int *dev)
{
    *dev = 0;
    return kOk;
}
int hipSetDevice(int dev)
{
    (void)dev;
    return kOk;
}
const char *hipGetErrorString(int e) { return e == kOutOfMemory ? "out of memory" : "error"; }
int hipGetLastError(void)
{
    const int e = g_error;
    g_error = kOk;
    return e;
}
int hipStreamSynchronize(void *s)
{
    (void)s;
    return kOk;
}
int hipMemcpy(void *d, const void *s, size_t n, int kind)
{
    (void)d, (void)s, (void)n, (void)kind;
    return kOk;
}
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st)
{
    (void)st;
    return hipMemcpy(d, s, n, kind);
}
int hipGetSymbolAddress(void **p, const void *sym)
{
    *p = (void *)sym;
    return kOk;
}
int hipFuncSetAttribute(const void *f, int attr, int value)
{
    (void)f, (void)attr, (void)value;
    return kOk;
}
int hipEventCreate(void **e)
{
    *e = (void *)1;
    return kOk;
}
int hipEventDestroy(void *e)
{
    (void)e;
    return kOk;
}
int hipEventRecord(void *e, void *s)
{
    (void)e, (void)s;
    return kOk;
}
int hipEventElapsedTime(float *ms, void *a, void *b)
{
    (void)a, (void)b;
    *ms = 0.f;
    return kOk;
}
void **__hipRegisterFatBinary(const void *data)
{
    static void *module;
    (void)data;
    return &module;
}
void __hipRegisterFunction(void **m, const void *f, char *df, const char *n, unsigned t, void *a, void *b, void *c,
                           void *d, int *w)
{
    (void)m, (void)f, (void)df, (void)n, (void)t, (void)a, (void)b, (void)c, (void)d, (void)w;
}
void __hipRegisterVar(void **m, void *v, char *h, char *dv, int e, size_t s, int c, int g)
{
    (void)m, (void)v, (void)h, (void)dv, (void)e, (void)s, (void)c, (void)g;
}
void __hipUnregisterFatBinary(void **m) { (void)m; }
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *s)
{
    (void)lds, (void)s;
    g_grid = grid;
    g_block = block;
    return kOk;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **s)
{
    *grid = g_grid;
    *block = g_block;
    *lds = 0;
    *s = NULL;
    return kOk;
}

int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *s)
{
    (void)lds, (void)s;
    Dl_info info;
    const char *name = dladdr(f, &info) && info.dli_sname ? info.dli_sname : "?";
    const int bad = (uint64_t)grid.x * block.x >> 32 || (uint64_t)grid.y * block.y >> 32 ||
                    (uint64_t)grid.z * block.z >> 32 || !grid.x || !grid.y || !grid.z;
    g_len += (size_t)snprintf(g_log + g_len, sizeof g_log - g_len, "%s %u %u %u %u%s\n", name, grid.x, grid.y, grid.z,
                              block.x, bad ? " refused" : "");
    if (bad)
        return g_error = kInvalidConfiguration;
    if (strstr(name, "k_compact")) { /* its outcome, as the kernel publishes it */
        uint64_t *r = *(uint64_t **)args[5];
        const uint64_t tag = (uint64_t) * (uint32_t *)args[6] << 32;
        r[0] = tag | g_flags;
        r[1] = tag | g_count;
        r[2] = tag | g_bucket;
    }
    return kOk;
}
