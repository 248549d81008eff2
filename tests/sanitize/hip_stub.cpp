// A host-only stand-in for the HIP runtime functions that the library and
// tests/c_caller_gpu.c call: device memory is host memory of the exact size,
// kernels do not run, and every handle is checked (a second free or destroy of
// anything aborts).  For runs of the host code under AddressSanitizer.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>

namespace {
std::mutex mu;
std::map<void*, size_t> memory;
std::set<void*> events, pools;
long launches = 0;

[[noreturn]] void die(const char* what) {
    std::fprintf(stderr, "hip stub: %s\n", what);
    std::abort();
}
void* get(size_t n) {
    void* p = std::malloc(n ? n : 1);
    std::lock_guard<std::mutex> lk(mu);
    memory[p] = n;
    return p;
}
void drop(void* p) {
    if (!p) return;
    std::lock_guard<std::mutex> lk(mu);
    if (!memory.erase(p)) die("freed memory that is not allocated");
    std::free(p);
}
void need(const std::set<void*>& s, void* h, const char* what) {
    std::lock_guard<std::mutex> lk(mu);
    if (!s.count(h)) die(what);
}
struct AtExit {
    ~AtExit() { std::fprintf(stderr, "hip stub: %ld launches, %zu allocations left\n", launches, memory.size()); }
} at_exit;
}  // namespace

extern "C" {
char __hip_fatbin[16];
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
    if (!grid.x || !grid.y || (size_t)grid.x * block.x >= (size_t(1) << 32)) die("a launch's grid");
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* shared, hipStream_t* stream) {
    *grid = *block = dim3(1);
    *shared = 0;
    *stream = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { ++launches; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 4; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static void* s = get(size_t(256) << 20); *p = s; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = get(n); return hipSuccess; }
hipError_t hipFree(void* p) { drop(p); return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { *p = get(n); return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void** p, size_t n, hipMemPool_t pool, hipStream_t) {
    need(pools, pool, "a pool that does not exist");
    *p = get(n);
    return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) { drop(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) {
    void* h = std::malloc(1);
    std::lock_guard<std::mutex> lk(mu);
    pools.insert(h);
    *p = static_cast<hipMemPool_t>(h);
    return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t p, hipMemPoolAttr, void*) { need(pools, p, "a pool that does not exist"); return hipSuccess; }
hipError_t hipMemPoolGetAttribute(hipMemPool_t p, hipMemPoolAttr, void* v) {
    need(pools, p, "a pool that does not exist");
    *static_cast<uint64_t*>(v) = 0;
    return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t p, size_t) { need(pools, p, "a pool that does not exist"); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    void* h = std::malloc(1);
    std::lock_guard<std::mutex> lk(mu);
    events.insert(h);
    *e = static_cast<hipEvent_t>(h);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) {
    std::lock_guard<std::mutex> lk(mu);
    if (!events.erase(e)) die("destroyed an event that does not exist");
    std::free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { need(events, e, "an event that does not exist"); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { need(events, e, "an event that does not exist"); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { need(events, e, "an event that does not exist"); return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t e, unsigned) { need(events, e, "an event that does not exist"); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
}
