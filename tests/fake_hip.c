/* A stand-in for the parts of the HIP runtime that the library calls, for
 * tests of its launch rules on a machine without a GPU.  "Device" memory is
 * host memory, kernels are not run: every launch is handed to a callback. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef void (*launch_cb)(const char *name, const uint32_t *grid_block, uint64_t lds, const void *args);

static launch_cb g_cb;
static struct { const void *fn; const char *name; } g_kernels[4096];
static int g_n;

void fake_hip_on_launch(launch_cb cb) { g_cb = cb; }

void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)d; (void)e; (void)s; (void)c; (void)g;
}
void __hipRegisterFunction(void **m, const void *fn, char *dev, const char *name, unsigned lim, void *a, void *b,
                           void *c, void *d, int *w)
{
    (void)m; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
    if (g_n < (int)(sizeof(g_kernels) / sizeof(g_kernels[0]))) {
        g_kernels[g_n].fn = fn;
        g_kernels[g_n++].name = name;
    }
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *s, void **st) { (void)g; (void)b; (void)s; (void)st; return 1; }

int hipLaunchKernel(const void *fn, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    (void)stream;
    const uint32_t gb[6] = {grid.x, grid.y, grid.z, block.x, block.y, block.z};
    for (int k = 0; k < g_n; ++k)
        if (g_kernels[k].fn == fn && g_cb)
            g_cb(g_kernels[k].name, gb, lds, args[0]);
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int dev) { (void)attr; (void)dev; *v = 256; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? 0 : 2; }
int hipFree(void *p) { free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return hipMalloc(p, n); }
int hipHostGetDevicePointer(void **d, void *h, unsigned f) { (void)f; *d = h; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = (void *)(uintptr_t)0x400000000000ull; return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }

/* Addresses from 2^46 on are pinned host memory, others device memory. */
typedef struct { int type, device; void *dev, *host; int managed; unsigned flags; } attr_t;
int hipPointerGetAttributes(attr_t *a, const void *p)
{
    memset(a, 0, sizeof(*a));
    a->type = (uintptr_t)p >> 46 ? 1 : 2;
    a->dev = (void *)p;
    return 0;
}
