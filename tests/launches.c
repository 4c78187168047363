/* A stand-in for the HIP runtime's launches, for tests without a GPU: "device" memory is host memory, kernels do nothing, and what was launched can be
 * asked for.  Refused as the runtime refuses it is a launch of 2^32 threads or more in a dimension, or of more than 65535 workgroups in y or z.  The
 * stream is in a capture when the test says so.  Preloaded before libmosaic. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
static struct { const void *f; char name[256]; } kernels[4096];
static struct { int kernel; dim3 g; } launched[1 << 16];
static int n_kernels, n_launched, last_error, capturing;
static char scratch[1 << 12];

/* the kernels' names, as the library registers them */
void __hipRegisterFunction(void **modules, const void *host, char *device, const char *name, unsigned limit, void *tid, void *bid, dim3 *block, dim3 *grid,
                           int *size) {
    (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)size;
    if (n_kernels == 4096) return;
    kernels[n_kernels].f = host;
    strncpy(kernels[n_kernels].name, name, sizeof kernels[0].name - 1);
    ++n_kernels;
}
/* (a launch's shape on its way from the caller to the kernel's stub) */
static struct { dim3 g, b; size_t lds; void *s; } call;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *s) { call.g = g; call.b = b; call.lds = lds; call.s = s; return 0; }
int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **s) { *g = call.g; *b = call.b; *lds = call.lds; *s = call.s; return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
    (void)args; (void)lds; (void)s;
    const uint64_t most = 1ull << 32;
    if ((uint64_t)g.x * b.x >= most || (uint64_t)g.y * b.y >= most || (uint64_t)g.z * b.z >= most || g.y > 65535 || g.z > 65535) return last_error = 9;
    int k = 0;
    while (k < n_kernels && kernels[k].f != f) ++k;
    if (n_launched < 1 << 16) { launched[n_launched].kernel = k; launched[n_launched].g = g; ++n_launched; }
    return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = scratch; return 0; }
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)p; (void)v; (void)n; (void)s; return 0; }
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing; return 0; }
int hipMemcpyWithStream(void *dst, const void *src, size_t n, int kind, void *s) { (void)kind; (void)s; memcpy(dst, src, n); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }

int launches(void) { return n_launched; }
const char *launch_name(int i) { return launched[i].kernel < n_kernels ? kernels[launched[i].kernel].name : ""; }
unsigned launch_grid(int i, int dim) { return dim == 0 ? launched[i].g.x : dim == 1 ? launched[i].g.y : launched[i].g.z; }
void forget_launches(void) { n_launched = 0; }
void set_capturing(int on) { capturing = on; }
