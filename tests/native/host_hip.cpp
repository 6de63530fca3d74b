// The HIP entry points that libpfac.so calls, over host memory and without a
// device: memory comes from malloc, kernels do not run.  Every call that
// allocates, clears, copies, launches or waits is written down, one a line, so
// that a test on the CPU sees what the library does around its kernels.  Loaded
// before libpfac.so into the global scope, it takes the place of the runtime.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>

namespace {

std::mutex mu;
std::string text;                          // the lines since the last clear
std::map<const void *, std::string> names;  // kernels by their host address
std::map<void *, size_t> sizes;            // live device allocations
size_t malloc_limit = ~(size_t)0;          // larger ones are refused
std::string refuse;                        // launches of kernels so named fail
bool capturing = false;
hipError_t last = hipSuccess;

void line(const char *fmt, unsigned long long a = 0, unsigned long long b = 0, unsigned long long c = 0,
          unsigned long long d = 0, const char *s = "") {
    char buf[512];
    std::snprintf(buf, sizeof buf, fmt, a, b, c, d, s);
    std::lock_guard<std::mutex> lock(mu);
    text += buf;
    text += '\n';
}

hipError_t fail(hipError_t e) {
    last = e;
    return e;
}

// the pending launch of the <<<>>> form
thread_local dim3 p_grid, p_block;
thread_local size_t p_lds;
thread_local hipStream_t p_stream;

}  // namespace

extern "C" {

// ---- for the tests
const char *host_hip_text() { return text.c_str(); }
void host_hip_clear() { text.clear(); }
void host_hip_limit(size_t bytes) { malloc_limit = bytes; }
void host_hip_refuse(const char *name) { refuse = name; }
void host_hip_capture(int on) { capturing = on != 0; }
// bytes of the device allocation that holds p, from p on (0: none does)
size_t host_hip_room(const void *p) {
    std::lock_guard<std::mutex> lock(mu);
    for (auto &a : sizes) {
        const char *lo = (const char *)a.first, *at = (const char *)p;
        if (at >= lo && at < lo + a.second) return (size_t)(lo + a.second - at);
    }
    return 0;
}

// ---- the runtime
void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {
    names[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    p_grid = grid;
    p_block = block;
    p_lds = lds;
    p_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = p_grid;
    *block = p_block;
    *lds = p_lds;
    *s = p_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **, size_t lds, hipStream_t s) {
    const std::string &n = names[fn];
    if (!refuse.empty() && n.find(refuse) != std::string::npos) return fail(hipErrorLaunchFailure);
    line("launch grid %llu block %llu lds %llu stream %llu %s", grid.x, block.x, lds, (unsigned long long)(uintptr_t)s,
         n.c_str());
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t n) {
    *p = n <= malloc_limit ? std::malloc(n) : nullptr;
    line(*p ? "malloc %llu" : "malloc refused %llu", n);
    if (!*p) return fail(hipErrorOutOfMemory);
    std::lock_guard<std::mutex> lock(mu);
    sizes[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    {
        std::lock_guard<std::mutex> lock(mu);
        sizes.erase(p);
    }
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    *p = std::calloc(1, n);
    line("host malloc %llu", n);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemset(void *p, int v, size_t n) {
    std::memset(p, v, n);
    line("memset %llu", n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *, const void *, size_t n, hipMemcpyKind, hipStream_t) {
    line("copy %llu", n);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    line("sync stream %llu", (unsigned long long)(uintptr_t)s);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    line("sync device");
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *) {
    static char *area = (char *)std::malloc(64u << 20);
    *p = area;
    return hipSuccess;
}

hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 * 1024 : 0;
    return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) {
    std::memset(a, 0, sizeof *a);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 1;
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)(uintptr_t)0x1000;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) {
    *c = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    capturing = true;
    line("capture begins");
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    capturing = false;
    *g = (hipGraph_t)(uintptr_t)0x2000;
    line("capture ends");
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *x = (hipGraphExec_t)(uintptr_t)0x3000;
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)(uintptr_t)0x4000;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventRecordWithFlags(hipEvent_t, hipStream_t, unsigned) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}

}  // extern "C"
