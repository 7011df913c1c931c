/* A HIP runtime without a device, for host-side tests: two "devices" of 256 CUs, device memory in host memory, kernels
 * that do nothing.  Launches, function attributes, event records and waits are printed to stdout, one a line. */
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static int dev = 0;
static dim3 cfg_grid, cfg_block;
static size_t cfg_lds;
static hipStream_t cfg_stream;

hipError_t hipGetDeviceCount(int *n) { *n = 2; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = dev; return hipSuccess; }
hipError_t hipSetDevice(int d) { dev = d; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(n ? n : 1, 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t t) { (void)t; return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void *d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { (void)e; return "fake"; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int d) { (void)a; (void)d; *v = 256; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int d) { (void)d; memset(p, 0, sizeof *p); p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = malloc(64); return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *f) { (void)f; memset(a, 0, sizeof *a); a->sharedSizeBytes = 256; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute a, int v) { (void)a; printf("allow %d %p %d\n", dev, f, v); return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l) { (void)f; (void)l; *n = b >= 512 ? 1 : 512 / b; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned f) { (void)f; *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { (void)s; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned f) { (void)f; *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { (void)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { printf("record %p %p\n", (void *)e, (void *)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned f) { (void)f; printf("wait %p %p\n", (void *)s, (void *)e); return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **a, size_t l, hipStream_t s) {
    (void)a;
    printf("launch %d %p %zu %p %u %u\n", dev, f, l, (void *)s, g.x, b.x);
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) { cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) { *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream; return hipSuccess; }
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *f, char *n, const char *d, unsigned t, void *a, void *b, void *c, void *e, int *w) { (void)h; (void)f; (void)n; (void)d; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w; }
void __hipRegisterVar(void **h, void *v, char *a, char *b, int c, size_t d, int e, int f) { (void)h; (void)v; (void)a; (void)b; (void)c; (void)d; (void)e; (void)f; }
