/* The HIP calls of the library's host code, on host memory: device memory with a limit, kernels that do nothing.  Loaded
   before the library (RTLD_GLOBAL), so that the host paths around the kernels can be tested without a GPU.  Every
   function returns hipSuccess (0) unless said otherwise. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

static size_t used, limit = (size_t)1 << 40;
static int allocations, launches, capturing, host_allocations, host_blocks, unsynchronized;
static uint64_t grid_xy;                        /* of the latest launch */
struct head { size_t bytes, pad[31]; };

void fake_set_limit(size_t bytes) { limit = bytes; }
size_t fake_used(void) { return used; }
int fake_allocations(void) { return allocations; }
int fake_host_allocations(void) { return host_allocations; }
int fake_host_blocks(void) { return host_blocks; }      /* page-locked, not freed */
void fake_fail_synchronize(int on) { unsynchronized = on; }
int fake_launches(void) { return launches; }
unsigned fake_grid(void) { return (unsigned)grid_xy; }

void fake_capture(int on) { capturing = on; }      /* 2: hipStreamIsCapturing has no answer */

int hipMalloc(void **p, size_t n) {
    struct head *h;
    ++allocations;
    if (used + n > limit || !(h = aligned_alloc(256, sizeof *h + ((n + 255) & ~(size_t)255)))) return 2;      /* hipErrorOutOfMemory */
    h->bytes = n;
    used += n;
    *p = h + 1;
    return 0;
}
int hipFree(void *p) {
    struct head *h = (struct head *)p - 1;
    if (p) { used -= h->bytes; free(h); }
    return 0;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
    (void)flags;
    if (!(*p = calloc(1, n))) return 2;
    ++host_allocations;
    ++host_blocks;
    return 0;
}
int hipHostFree(void *p) { if (p) --host_blocks; free(p); return 0; }
int hipHostGetDevicePointer(void **d, void *h, unsigned flags) { (void)flags; *d = h; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *stream) { (void)kind; (void)stream; memcpy(d, s, n); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; memcpy(d, s, n); return 0; }
int hipMemsetAsync(void *d, int v, size_t n, void *stream) { (void)stream; memset(d, v, n); return 0; }
int hipGetSymbolAddress(void **p, const void *symbol) { static _Alignas(256) uint8_t scratch[4 << 20]; (void)symbol; *p = scratch; return 0; }
int hipLaunchKernel(const void *f, uint64_t gxy, uint32_t gz, uint64_t bxy, uint32_t bz, void **args, size_t lds, void *stream) {
    (void)f; (void)gxy; (void)gz; (void)bxy; (void)bz; (void)args; (void)lds; (void)stream;
    ++launches;
    return 0;
}
int __hipPushCallConfiguration(uint64_t gxy, uint32_t gz, uint64_t bxy, uint32_t bz, size_t lds, void *stream) {
    (void)gz; (void)bxy; (void)bz; (void)lds; (void)stream;
    grid_xy = gxy;
    return 0;
}
int __hipPopCallConfiguration(void *grid, void *block, size_t *lds, void **stream) {
    memset(grid, 0, 12); memset(block, 0, 12); *lds = 0; *stream = NULL;
    return 0;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int d) { return d == 0 ? 0 : 101; }      /* hipErrorInvalidDevice */
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int e) { return e == 2 ? "out of memory" : "error"; }
int hipDeviceSynchronize(void) { return unsynchronized ? 906 : 0; }
int hipStreamSynchronize(void *s) { (void)s; return 0; }
int hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; *s = NULL; return 0; }
int hipStreamDestroy(void *s) { (void)s; return 0; }
int hipStreamWaitEvent(void *s, void *e, unsigned f) { (void)s; (void)e; (void)f; return 0; }
int hipEventCreateWithFlags(void **e, unsigned f) { (void)f; *e = NULL; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipStreamIsCapturing(void *s, int *status) { (void)s; *status = capturing == 1; return capturing == 2 ? 906 : 0; }      /* hipErrorStreamCaptureImplicit */
