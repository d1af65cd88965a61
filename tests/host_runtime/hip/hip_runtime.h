// A stand-in for the HIP runtime on the host, for tests of the library's host
// code without a GPU: "device" memory is host memory, work runs when it is
// enqueued, and streams and events remember the device that was current when
// they were made (an event may be recorded only on a stream of its own device).
#pragma once

#include <atomic>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>

#define __device__
#define __align__(n) alignas(n)
#define HIP_SYMBOL(x) (&(x))

enum hipError_t {
    hipSuccess = 0,
    hipErrorInvalidValue = 1,
    hipErrorOutOfMemory = 2,
    hipErrorInvalidHandle = 400
};
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal = 1 };
constexpr unsigned hipStreamNonBlocking = 1, hipEventDisableTiming = 2;
constexpr unsigned hipEventReleaseToSystem = 0x40000000, hipHostMallocCoherent = 0x40000000;

struct FakeStream { int device; };
struct FakeEvent { int device; double at; };
struct FakeGraph {};
typedef FakeStream* hipStream_t;
typedef FakeEvent* hipEvent_t;
typedef FakeGraph* hipGraph_t;
typedef FakeGraph* hipGraphExec_t;

namespace fake {
inline thread_local int device = 0;               // current device of the thread
inline std::atomic<int> pinned_allocs{0}, pinned_live{0}, events_live{0}, foreign_events{0};
inline std::atomic<int> event_records{0}, device_copies{0};
inline bool no_pinned = false;                    // hipHostMalloc fails
inline std::atomic<int> last_error{0};
inline double now_ms = 0.0;                       // time of the timed work
inline std::function<void()> on_wait;             // before a wait for an event returns
}  // namespace fake

inline const char* hipGetErrorString(hipError_t e) { return e == hipSuccess ? "success" : "error"; }
inline hipError_t hipGetLastError() { return (hipError_t)fake::last_error.exchange(0); }
inline hipError_t hipGetDevice(int* d) { *d = fake::device; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { fake::device = d; return hipSuccess; }
inline hipError_t hipMalloc(void** p, size_t n) {
    *p = std::calloc(1, n);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (fake::no_pinned) {
        fake::last_error = hipErrorOutOfMemory;
        return hipErrorOutOfMemory;
    }
    ++fake::pinned_allocs;
    ++fake::pinned_live;
    return hipMalloc(p, n);
}
inline hipError_t hipHostFree(void* p) {
    if (p) --fake::pinned_live;
    return hipFree(p);
}
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    if (k == hipMemcpyHostToDevice) ++fake::device_copies;
    std::memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(d, s, n, k);
}
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = new FakeStream{fake::device};
    return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) { delete s; return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = new FakeEvent{fake::device, 0.0};
    ++fake::events_live;
    return hipSuccess;
}
inline hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
inline hipError_t hipEventDestroy(hipEvent_t e) {
    --fake::events_live;
    delete e;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    ++fake::event_records;
    if (s && e->device != s->device) {
        ++fake::foreign_events;
        return hipErrorInvalidHandle;
    }
    e->at = fake::now_ms;
    return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t) {
    if (fake::on_wait) fake::on_wait();
    return hipSuccess;
}
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(b->at - a->at);
    return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { *g = nullptr; return hipSuccess; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t* g, hipGraph_t, void*, void*, size_t) {
    *g = nullptr;
    return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
template <class T>
hipError_t hipGetSymbolAddress(void** p, T* symbol) {
    *p = (void*)symbol;
    return hipSuccess;
}
