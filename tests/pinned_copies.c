/* A stand-in for the HIP runtime calls of a large read-back, for tests without a GPU: "device" memory is host memory, kernels do
 * nothing, and an asynchronous copy is done when an event recorded after it is waited for, not before.  Memory that another copy is still to
 * fill is never handed a second one.  Preloaded before libmosaic. */
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
static struct { void *dst; const void *src; size_t n; int done; } q[1 << 16];
static int n_q, max_open, events[64], n_events;
static char scratch[1 << 12];
static int fail_at = -1;

int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = scratch; return 0; }
int hipGetLastError(void) { return 0; }
int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
    (void)f; (void)g; (void)b; (void)args; (void)lds; (void)s;
    return 0;
}
int hipMemsetAsync(void *p, int v, size_t n, void *s) { (void)s; memset(p, v, n); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned flags) { (void)flags; *p = malloc(n); memset(*p, 0xee, n); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { (void)flags; *e = &events[n_events++]; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipMemcpyAsync(void *dst, const void *src, size_t n, int kind, void *s) {
    (void)kind; (void)s;
    if (n_q == fail_at) return 1;
    int open = 0;
    for (int i = 0; i < n_q; ++i)
        if (!q[i].done) { ++open; if (q[i].dst == dst) abort(); }
    if (open + 1 > max_open) max_open = open + 1;
    q[n_q].dst = dst; q[n_q].src = src; q[n_q].n = n; q[n_q].done = 0;
    ++n_q;
    return 0;
}
int hipEventRecord(void *e, void *s) { (void)s; *(int *)e = n_q; return 0; }
int hipEventSynchronize(void *e) {
    for (int i = 0; i < *(int *)e; ++i)
        if (!q[i].done) { memcpy(q[i].dst, q[i].src, q[i].n); q[i].done = 1; }
    return 0;
}
int hipMemcpyWithStream(void *dst, const void *src, size_t n, int kind, void *s) {
    (void)kind; (void)s;
    memcpy(dst, src, n);
    return 0;
}
int most_open(void) { const int m = max_open; max_open = 0; return m; }
int copies(void) { const int n = n_q; n_q = 0; return n; }
void fail_copy(int i) { fail_at = i; }
