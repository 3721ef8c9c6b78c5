// A stand-in for the HIP runtime, linked in front of it: device memory is host
// memory that starts as zeros, kernels do nothing, streams only count what was
// queued on them.  With it the host code of libhyperim.so runs without a GPU,
// allocations can be made to fail, and the order of locks, waits and queued
// work can be checked.  Kernels write nothing, so every RR set comes out empty
// and every count zero.
#include "fake_hip.h"

#include <hip/hip_runtime_api.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>
#include <unistd.h>

#include <algorithm>
#include <map>
#include <mutex>
#include <utility>

namespace fake {
std::atomic<size_t> total{288ull << 30}, used{0}, peak{0};
std::atomic<long> mallocs{0}, fail_from{-1}, launches{0}, device_syncs{0}, overlaps{0};
std::atomic<bool> watch{false}, stalled{false};
std::atomic<long> blocked{0};
std::atomic<int> sync_us{0};
std::atomic<void (*)()> on_device_sync{nullptr};
}  // namespace fake

namespace {
std::mutex mu;
std::map<void *, size_t> blocks;
std::map<hipStream_t, long> pending;   // work queued since the stream was last waited for
std::map<hipEvent_t, std::pair<hipStream_t, long>> recorded;

hipError_t queued(hipStream_t s) {
    std::lock_guard<std::mutex> l(mu);
    if (fake::watch)
        for (const auto &p : pending)
            if (p.first != s && p.second > 0) ++fake::overlaps;
    ++pending[s];
    return hipSuccess;
}
void pause_us(int us) {
    if (us > 0) usleep((useconds_t)us);
}
struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
thread_local Config config;
}  // namespace

size_t fake::live_blocks() {
    std::lock_guard<std::mutex> l(mu);
    return blocks.size();
}
bool fake::live(const void *p) {
    std::lock_guard<std::mutex> l(mu);
    return blocks.count(const_cast<void *>(p)) != 0;
}

#define FAKE extern "C" __attribute__((visibility("default")))

FAKE hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s) {
    config = {g, b, sh, s};
    return hipSuccess;
}
FAKE hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *sh, hipStream_t *s) {
    *g = config.grid;
    *b = config.block;
    *sh = config.shared;
    *s = config.stream;
    return hipSuccess;
}
FAKE void **__hipRegisterFatBinary(const void *) {
    static void *handle;
    return &handle;
}
FAKE void __hipUnregisterFatBinary(void **) {}
FAKE void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned int, void *, void *, void *,
                                void *, int *) {}
FAKE void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

FAKE hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t s) {
    ++fake::launches;
    return queued(s);
}
FAKE hipError_t hipExtLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t s, hipEvent_t, hipEvent_t,
                                   int) {
    ++fake::launches;
    return queued(s);
}

FAKE hipError_t hipMalloc(void **p, size_t n) {
    const long i = fake::mallocs++;
    const long from = fake::fail_from;
    std::lock_guard<std::mutex> l(mu);
    if ((from >= 0 && i >= from) || fake::used + n > fake::total) return hipErrorOutOfMemory;
    void *m = mmap(nullptr, n ? n : 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (m == MAP_FAILED) return hipErrorOutOfMemory;
    blocks[m] = n;
    fake::used += n;
    if (fake::used > fake::peak) fake::peak = fake::used.load();
    *p = m;
    return hipSuccess;
}
FAKE hipError_t hipFree(void *p) {
    std::lock_guard<std::mutex> l(mu);
    if (!p) return hipSuccess;
    auto it = blocks.find(p);
    if (it == blocks.end()) return hipErrorInvalidValue;
    fake::used -= it->second;
    munmap(p, it->second ? it->second : 1);
    blocks.erase(it);
    return hipSuccess;
}
FAKE hipError_t hipHostMalloc(void **p, size_t n, unsigned int) {
    *p = calloc(1, n ? n : 1);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
FAKE hipError_t hipHostFree(void *p) {
    free(p);
    return hipSuccess;
}
FAKE hipError_t hipMemGetInfo(size_t *free_b, size_t *total_b) {
    *free_b = fake::total - fake::used;
    *total_b = fake::total;
    return hipSuccess;
}
FAKE hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t s) {
    memmove(dst, src, n);
    return queued(s);
}
// (all that the library sets is set to zero, and is zero from the start)
FAKE hipError_t hipMemsetAsync(void *, int, size_t, hipStream_t s) { return queued(s); }
FAKE hipError_t hipMemset(void *, int, size_t) { return hipSuccess; }

FAKE hipError_t hipStreamSynchronize(hipStream_t s) {
    {
        std::lock_guard<std::mutex> l(mu);
        if (pending[s] == 0) return hipSuccess;
    }
    if (fake::stalled) ++fake::blocked;
    pause_us(fake::sync_us);
    std::lock_guard<std::mutex> l(mu);
    pending[s] = 0;
    return hipSuccess;
}
FAKE hipError_t hipDeviceSynchronize() {
    ++fake::device_syncs;
    if (void (*f)() = fake::on_device_sync) f();
    std::lock_guard<std::mutex> l(mu);
    for (auto &p : pending) p.second = 0;
    return hipSuccess;
}
FAKE hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
    *s = reinterpret_cast<hipStream_t>(malloc(1));
    return hipSuccess;
}
FAKE hipError_t hipStreamDestroy(hipStream_t s) {
    std::lock_guard<std::mutex> l(mu);
    pending.erase(s);
    free(s);
    return hipSuccess;
}
FAKE hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
FAKE hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
FAKE hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    return hipErrorNotSupported;
}
FAKE hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
FAKE hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
FAKE hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }

FAKE hipError_t hipEventCreate(hipEvent_t *e) {
    *e = reinterpret_cast<hipEvent_t>(malloc(1));
    return hipSuccess;
}
FAKE hipError_t hipEventDestroy(hipEvent_t e) {
    free(e);
    return hipSuccess;
}
FAKE hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    const hipError_t rc = queued(s);
    std::lock_guard<std::mutex> l(mu);
    recorded[e] = {s, pending[s]};
    return rc;
}
FAKE hipError_t hipEventQuery(hipEvent_t) { return fake::stalled ? hipErrorNotReady : hipSuccess; }
FAKE hipError_t hipEventSynchronize(hipEvent_t e) {   // the work before the event is done
    hipStream_t s;
    {
        std::lock_guard<std::mutex> l(mu);
        s = recorded[e].first;
        if (pending[s] == 0) return hipSuccess;
    }
    pause_us(fake::sync_us);
    std::lock_guard<std::mutex> l(mu);
    pending[s] -= std::min(pending[s], recorded[e].second);
    recorded[e].second = 0;
    return hipSuccess;
}
FAKE hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 0.f;
    return hipSuccess;
}

FAKE hipError_t hipGetDevice(int *d) {
    *d = 0;
    return hipSuccess;
}
FAKE hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    *v = 256;   // compute units
    return hipSuccess;
}
FAKE hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int) {
    memset(p, 0, sizeof(*p));
    return hipSuccess;
}
FAKE int hipGetStreamDeviceId(hipStream_t) { return 0; }
FAKE hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidSymbol; }
FAKE hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
    *n = 6;
    return hipSuccess;
}
FAKE hipError_t hipGetLastError() { return hipSuccess; }
FAKE const char *hipGetErrorString(hipError_t) { return "stand-in runtime"; }
