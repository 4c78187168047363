/* A stand-in for the HIP runtime calls that the observers make, for tests without a GPU: "device" memory is host memory,
 * kernels do nothing, and an asynchronous copy to or from pageable memory is late -- it is done when the runtime says so
 * (late_copies_finish), not when its stream is synchronised, which is all that the runtime's documentation leaves open.
 * Host memory counts as pageable throughout.  Preloaded before libmosaic. */
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
static struct { void *dst; const void *src; size_t n; } late[4096];
static int n_late;
static size_t n_bytes;
static char scratch[1 << 12];

int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = scratch; return 0; }
int hipGetLastError(void) { return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
    (void)f; (void)g; (void)b; (void)args; (void)lds; (void)s;
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)s; memset(p, v, n); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *s) {
    (void)kind; (void)s;
    if (n_late == 4096) abort();
    late[n_late].dst = dst; late[n_late].src = src; late[n_late].n = n;
    ++n_late;
    return 0;
}
int hipMemcpyWithStream(void *dst, const void *src, size_t n, int kind, void *s) {
    (void)kind; (void)s;
    memcpy(dst, src, n);
    n_bytes += n;
    return 0;
}
/* how many copies are still to be done, and the bytes that others have copied since the last time */
int late_copies_pending(void) { return n_late; }
size_t copied_bytes(void) { const size_t n = n_bytes; n_bytes = 0; return n; }
