// A HIP runtime without a GPU, for tests of what the library does on the host: device memory is numbers, work is a list.
#include <hip/hip_runtime_api.h>

#include <map>
#include <mutex>
#include <string>

namespace {
std::recursive_mutex lock;
struct State {
    std::map<char*, size_t> memory;
    size_t limit = 0, used = 0;
    char* next = reinterpret_cast<char*>((size_t)1 << 40);
    bool capturing = false, broken = false;                // a stream is being captured; a call has spoilt that
    int device = 0;
    std::string events, launches;
    std::map<const void*, std::string> kernels;
} g;
hipError_t note(const char* what) {
    std::lock_guard<std::recursive_mutex> guard(lock);
    g.events += what;
    g.events += ' ';
    return hipSuccess;
}
}  // namespace

extern "C" {
void fake_reset(size_t limit) {
    g.limit = limit;
    g.capturing = g.broken = false;
    g.device = 0;
    g.events.clear();
}
void fake_capture(int on) { g.capturing = on != 0; }
int fake_broken() { return g.broken; }
void fake_device(int device) { g.device = device; }
size_t fake_used() { return g.used; }
const char* fake_launches() {                         // names of the kernels since the last call
    static std::string out;
    out.swap(g.launches);
    g.launches.clear();
    return out.c_str();
}
const char* fake_events() {
    static std::string out;
    out.swap(g.events);
    g.events.clear();
    return out.c_str();
}

hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::recursive_mutex> guard(lock);
    if (g.capturing) return hipErrorStreamCaptureUnsupported;
    if (n > g.limit || g.used > g.limit - n) return hipErrorOutOfMemory;
    *p = g.next;
    g.memory[g.next] = n;
    g.next += (n + 4095) / 4096 * 4096;
    g.used += n;
    return note("malloc");
}
hipError_t hipFree(void* p) {
    std::lock_guard<std::recursive_mutex> guard(lock);
    const auto at = g.memory.find(static_cast<char*>(p));
    if (at == g.memory.end()) {
        note("wild-free");
        return hipErrorInvalidValue;
    }
    g.used -= at->second;
    g.memory.erase(at);
    return note("free");
}
hipError_t hipMemGetInfo(size_t* free, size_t* total) {
    std::lock_guard<std::recursive_mutex> guard(lock);
    *total = g.limit;
    *free = g.used > g.limit ? 0 : g.limit - g.used;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
    if (!g.capturing) return note("sync");
    g.broken = true;
    return hipErrorStreamCaptureUnsupported;
}
hipError_t hipMemsetAsync(void* p, int, size_t n, hipStream_t) {
    std::lock_guard<std::recursive_mutex> guard(lock);
    auto at = g.memory.upper_bound(static_cast<char*>(p));
    if (at == g.memory.begin() || (--at)->first + at->second < static_cast<char*>(p) + n) note("wild-write");
    return note("set");
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) { return note("copy"); }
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t, hipStream_t) {
    std::lock_guard<std::recursive_mutex> guard(lock);
    g.launches += g.kernels[kernel] + ' ';
    return note("launch");
}
hipError_t hipLaunchCooperativeKernel(const void*, dim3, dim3, void**, unsigned, hipStream_t) { return note("launch"); }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetDevice(int* device) {
    *device = g.device;
    return hipSuccess;
}
hipError_t hipSetDevice(int device) {
    g.device = device;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = reinterpret_cast<void*>((size_t)1 << 39);
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 1;
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = *block = dim3(1);
    *lds = 0;
    *s = nullptr;
    return hipSuccess;
}
void* __hipRegisterFatBinary(const void*) {
    static void* handle[2];
    return handle;
}
void __hipUnregisterFatBinary(void*) {}
void __hipRegisterFunction(void*, const void* kernel, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { g.kernels[kernel] = name; }
void __hipRegisterVar(void*, void*, char*, char*, int, size_t, int, int) {}
}
