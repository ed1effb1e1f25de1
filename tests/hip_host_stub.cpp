// The HIP calls of libdv's host side over plain memory, with no device: kernels
// are not run, only noted.  A test loads it with global symbols before the
// library, so that it can make a chosen call fail.
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "dv_internal.h"

static std::map<const void *, std::string> g_name;
static std::vector<int> g_headers;   // DV_PG_PAR of the first entry of each k_place
static int g_fail_record, g_stale_error;
static dim3 g_grid, g_block;
static size_t g_shmem;
static hipStream_t g_stream;

extern "C" {
void stub_fail_record(int n) { g_fail_record = n; }    // the next n records fail
void stub_stale_error(int n) { g_stale_error = n; }    // the next n hipGetLastError report one
int stub_headers(int *out, int cap) {
    for (int i = 0; i < (int)g_headers.size() && i < cap; ++i) out[i] = g_headers[i];
    return (int)g_headers.size();
}

void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *) { g_name[f] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
    g_grid = g; g_block = b; g_shmem = m; g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *m, hipStream_t *s) {
    *g = g_grid; *b = g_block; *m = g_shmem; *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3, dim3, void **args, size_t, hipStream_t) {
    if (g_name[f].find("k_place") != std::string::npos)
        g_headers.push_back(DV_PG_PAR(static_cast<const Batch *>(args[1])->pslot[0]));
    return hipSuccess;
}
hipError_t hipGetLastError() { return g_stale_error > 0 ? (--g_stale_error, hipErrorUnknown) : hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorUnknown; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetD32Async(hipDeviceptr_t d, int v, size_t n, hipStream_t) {
    for (size_t i = 0; i < n; ++i) static_cast<int *>(d)[i] = v;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(malloc(1)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(malloc(1)); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return g_fail_record > 0 ? (--g_fail_record, hipErrorUnknown) : hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
}
