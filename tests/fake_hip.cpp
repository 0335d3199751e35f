// A HIP runtime of two devices in host memory, for tests of the library's host
// code without a GPU: loaded (RTLD_GLOBAL) before the library, its calls take
// the place of the runtime's.  Device and page-locked memory are ordinary
// allocations that it keeps a list of; copies are queued per stream and done
// when the stream is waited for; kernels do nothing.  The test reads what was
// called (fake_*) and sets limits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace {
std::mutex mu;
std::atomic<bool> no_memory{false};
thread_local int inside = 0;   // this runtime's own allocations always succeed
struct Lock {
    std::lock_guard<std::mutex> lk{mu};
    Lock() { ++inside; }
    ~Lock() { --inside; }
};
struct Mem {
    size_t bytes;
    bool device;
    int at;
};
std::map<uintptr_t, Mem> mems;
struct Copy {
    void *dst;
    const void *src;
    size_t bytes;
};
std::map<hipStream_t, std::vector<Copy>> queued;
std::map<std::string, long> calls;
thread_local int current = 0;
size_t held = 0, peak = 0, limit = SIZE_MAX, copied_to_pageable = 0;
long fail_copy = -1;      // this many more copies succeed
std::atomic<long> not_ready{0};   // this many event queries say so
bool on_wrong = false;    // a call for another device than `expected`
int expected = -1;
char symbol[64 << 20];    // device variables

const Mem *find(const void *p) {
    auto it = mems.upper_bound((uintptr_t)p);
    if (it == mems.begin()) return nullptr;
    --it;
    return (uintptr_t)p < it->first + it->second.bytes ? &it->second : nullptr;
}
void note(const char *name, bool device_call = false) {
    ++calls[name];
    if (device_call && expected >= 0 && current != expected) on_wrong = true;
}
hipError_t get(void **p, size_t n, bool device, const char *name) {
    Lock lk;
    note(name, true);
    *p = nullptr;
    if (device && (n > limit || held > limit - n)) return hipErrorOutOfMemory;
    if (posix_memalign(p, 4096, std::max<size_t>(n, 1))) return hipErrorOutOfMemory;
    mems[(uintptr_t)*p] = Mem{std::max<size_t>(n, 1), device, current};
    if (device) peak = std::max(peak, held += n);
    return hipSuccess;
}
hipError_t drop(void *p, const char *name) {
    Lock lk;
    note(name);
    if (!p) return hipSuccess;
    auto it = mems.find((uintptr_t)p);
    if (it == mems.end()) return hipErrorInvalidValue;
    if (it->second.device) held -= it->second.bytes;
    mems.erase(it);
    std::free(p);
    return hipSuccess;
}
void run(hipStream_t s) {
    for (auto &c : queued[s]) std::memcpy(c.dst, c.src, c.bytes);
    queued[s].clear();
}
}  // namespace

void *operator new(size_t n) {
    void *p = no_memory && !inside ? nullptr : std::malloc(std::max<size_t>(n, 1));
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

static std::atomic<unsigned> cpus{16};
// std::thread::hardware_concurrency
extern "C" unsigned fake_hardware_concurrency() __asm__("_ZNSt6thread20hardware_concurrencyEv");
unsigned fake_hardware_concurrency() { return cpus; }

extern "C" {
// what the tests read and set
long fake_calls(const char *name) {
    Lock lk;
    return calls[name];
}
void fake_reset() {
    Lock lk;
    calls.clear();
    on_wrong = false;
    peak = held;
    copied_to_pageable = 0;
}
size_t fake_held() { return held; }
size_t fake_peak() { return peak; }
void fake_limit(size_t bytes) { limit = bytes; }
void fake_fail_copy(long after) { fail_copy = after; }
void fake_not_ready(long n) { not_ready = n; }
void fake_cpus(unsigned n) { cpus = n; }
void fake_no_memory(int on) { no_memory = on != 0; }   // host allocations (operator new) fail
void fake_expect_device(int d) { expected = d; }
int fake_on_wrong_device() { return on_wrong; }
void fake_set_current(int d) { current = d; }
size_t fake_bytes_to_pageable() { return copied_to_pageable; }
size_t fake_pending() {
    Lock lk;
    size_t n = 0;
    for (auto &q : queued) n += q.second.size();
    return n;
}
void *fake_pinned(size_t n) {
    void *p;
    return get(&p, n, false, "test") == hipSuccess ? p : nullptr;
}

hipError_t hipGetDeviceCount(int *n) { *n = 2; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = symbol; return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = (size_t)64 << 30; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return get(p, n, true, "hipMalloc"); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return get(p, n, false, "hipHostMalloc"); }
hipError_t hipFree(void *p) { return drop(p, "hipFree"); }
hipError_t hipHostFree(void *p) { return drop(p, "hipHostFree"); }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
    Lock lk;
    std::memset(a, 0, sizeof(*a));
    const Mem *m = find(p);
    a->type = m ? (m->device ? hipMemoryTypeDevice : hipMemoryTypeHost) : hipMemoryTypeUnregistered;
    a->device = m ? m->at : 0;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)std::malloc(16);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { std::free((void *)s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
    Lock lk;
    note("hipStreamSynchronize");
    run(s);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s) {
    Lock lk;
    note("hipMemcpyAsync");
    if (fail_copy == 0) return hipErrorInvalidValue;
    if (fail_copy > 0) --fail_copy;
    if (!find(dst)) copied_to_pageable += n;
    queued[s].push_back(Copy{dst, src, n});
    return hipSuccess;
}
hipError_t hipMemcpy2DAsync(void *dst, size_t dp, const void *src, size_t sp, size_t w, size_t h, hipMemcpyKind,
                            hipStream_t s) {
    Lock lk;
    for (size_t y = 0; y < h; ++y) queued[s].push_back(Copy{(char *)dst + y * dp, (const char *)src + y * sp, w});
    return hipSuccess;
}
hipError_t hipMemcpy(void *dst, const void *src, size_t n, hipMemcpyKind) {
    Lock lk;
    note("hipMemcpy");
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)std::calloc(1, 16); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { *(hipStream_t *)e = s; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) {
    Lock lk;
    run(*(hipStream_t *)e);
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    if (not_ready > 0) {
        --not_ready;
        return hipErrorNotReady;
    }
    return hipEventSynchronize(e);
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.0f; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
thread_local struct { dim3 grid, block; size_t lds; hipStream_t s; } config;
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    config = {grid, block, lds, s};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *s = config.s;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3 block, void **, size_t, hipStream_t) {
    Lock lk;
    note("hipLaunchKernel", true);
    if (block.x == 512) note("512 threads");
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = (hipGraph_t)std::malloc(8); return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    *e = (hipGraphExec_t)std::malloc(8);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { std::free((void *)g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { std::free((void *)e); return hipSuccess; }
}
