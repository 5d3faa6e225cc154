/* Stands in for the HIP runtime where a plan's arrays are uploaded: device memory is host memory within a budget, copies are
 * copies, kernels do nothing.  What a plan does when the device has no room can then be seen without one. */
#define _GNU_SOURCE
#include <malloc.h>
#include <stddef.h>
#include <stdlib.h>
#include <string.h>

static size_t live, budget = (size_t)-1, peak;

void stub_budget(size_t bytes) { budget = bytes; peak = live; }
size_t stub_live(void) { return live; }
size_t stub_peak(void) { return peak; }

static int take(void **p, size_t bytes) {
    *p = NULL;
    if (bytes > budget || live > budget - bytes) return 2; /* hipErrorOutOfMemory */
    size_t *block = calloc(1, bytes + 64);
    if (!block) return 2;
    *block = bytes;
    *p = (char *)block + 64;
    live += bytes;
    if (live > peak) peak = live;
    return 0;
}
static int give(void *p) {
    if (!p) return 0;
    size_t *block = (size_t *)((char *)p - 64);
    live -= *block;
    free(block);
    return 0;
}

int hipMalloc(void **p, size_t bytes) { return take(p, bytes); }
int hipFree(void *p) { return give(p); }
int hipHostMalloc(void **p, size_t bytes, unsigned flags) { (void)flags; *p = malloc(bytes); return *p ? 0 : 2; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemcpyAsync(void *dst, const void *src, size_t bytes, int kind, void *stream) { (void)kind; (void)stream; memcpy(dst, src, bytes); return 0; }
int hipMemsetAsync(void *dst, int value, size_t bytes, void *stream) { (void)stream; memset(dst, value, bytes); return 0; }
int hipStreamCreateWithFlags(void **s, unsigned flags) { (void)flags; *s = malloc(1); return 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipEventCreateWithFlags(void **e, unsigned flags) { (void)flags; *e = malloc(1); return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventDestroy(void *e) { free(e); return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }

typedef struct { unsigned x, y, z; } dim3_t;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shared, void *stream) { (void)grid; (void)block; (void)shared; (void)stream; return 0; }
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *shared, void **stream) {
    grid->x = grid->y = grid->z = block->x = block->y = block->z = 1;
    *shared = 0;
    *stream = NULL;
    return 0;
}
int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t shared, void *stream) {
    (void)f; (void)grid; (void)block; (void)args; (void)shared; (void)stream;
    return 0;
}
