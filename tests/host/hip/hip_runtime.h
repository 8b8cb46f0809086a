// Stand-in for the HIP runtime, for CPU tests of the library's host code
// (fh_runtime.cpp): "device" memory is host memory, copies happen at once and
// a captured graph counts its launches.  Failures follow ROCm 7: the error of
// a failed call stays until hipGetLastError() takes it, whatever succeeds in
// between, and a kernel launch reports it.  Counters are relaxed atomics, so
// that they order nothing between the threads of a test.
#pragma once

#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>

#define __host__
#define __device__
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (&(x))

struct int2 { int x, y; };
struct int4 { int x, y, z, w; };
struct uint2 { unsigned x, y; };

enum hipError_t {
    hipSuccess = 0,
    hipErrorInvalidValue = 1,
    hipErrorOutOfMemory = 2,
    hipErrorNotReady = 600,
    hipErrorStreamCaptureUnsupported = 900
};
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal };
constexpr unsigned hipHostMallocDefault = 0, hipEventDisableTiming = 2, hipStreamNonBlocking = 1;

typedef struct FakeStream *hipStream_t;
typedef struct FakeEvent *hipEvent_t;
typedef struct FakeGraph *hipGraph_t;
typedef struct FakeGraph *hipGraphExec_t;

struct hipDeviceProp_t {
    char gcnArchName[64];
    int multiProcessorCount;
};

namespace fake {
inline thread_local hipError_t last_error = hipSuccess;
inline std::atomic<int64_t> used{0}, limit{INT64_MAX};          // device memory
inline std::atomic<int64_t> pinned{0}, pinned_limit{INT64_MAX};  // pinned host memory
inline std::atomic<int> graphs{0};                               // graphs instantiated
// a capture under way: on another thread, where hipMalloc and hipFree are
// harmless and hipDeviceSynchronize breaks it, or on this one, where all three do
inline std::atomic<bool> capturing_elsewhere{false}, capturing_here{false};
inline std::atomic<int> captures_broken{0};

inline hipError_t fail(hipError_t e) { return last_error = e; }
inline hipError_t in_capture(bool elsewhere) {
    if (!capturing_here.load(std::memory_order_relaxed) &&
        !(elsewhere && capturing_elsewhere.load(std::memory_order_relaxed)))
        return hipSuccess;
    captures_broken.fetch_add(1, std::memory_order_relaxed);
    return fail(hipErrorStreamCaptureUnsupported);
}

// blocks carry their size in front
inline hipError_t alloc(void **p, size_t n, std::atomic<int64_t> &sum, std::atomic<int64_t> &most) {
    if (sum.load(std::memory_order_relaxed) + (int64_t)n > most.load(std::memory_order_relaxed)) {
        *p = nullptr;
        return fail(hipErrorOutOfMemory);
    }
    sum.fetch_add((int64_t)n, std::memory_order_relaxed);
    char *q = (char *)std::calloc(1, n + 64);
    std::memcpy(q, &n, sizeof n);
    *p = q + 64;
    return hipSuccess;
}
inline void release(void *p, std::atomic<int64_t> &sum) {
    if (!p) return;
    size_t n;
    std::memcpy(&n, (char *)p - 64, sizeof n);
    sum.fetch_sub((int64_t)n, std::memory_order_relaxed);
    std::free((char *)p - 64);
}
}  // namespace fake

inline hipError_t hipGetLastError() {
    const hipError_t e = fake::last_error;
    fake::last_error = hipSuccess;
    return e;
}
inline const char *hipGetErrorString(hipError_t e) { return e == hipErrorOutOfMemory ? "out of memory" : "error"; }

inline hipError_t hipMalloc(void **p, size_t n) {
    const hipError_t e = fake::in_capture(false);
    return e != hipSuccess ? e : fake::alloc(p, n, fake::used, fake::limit);
}
template <typename T>
hipError_t hipMalloc(T **p, size_t n) { return hipMalloc((void **)p, n); }
inline hipError_t hipFree(void *p) {
    const hipError_t e = fake::in_capture(false);
    if (e != hipSuccess) return e;
    fake::release(p, fake::used);
    return hipSuccess;
}
inline hipError_t hipHostMalloc(void **p, size_t n, unsigned) {
    return fake::alloc(p, n, fake::pinned, fake::pinned_limit);
}
inline hipError_t hipHostFree(void *p) {
    fake::release(p, fake::pinned);
    return hipSuccess;
}
inline hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) {
    return hipMemcpy(d, s, n, k);
}
inline hipError_t hipMemset(void *d, int v, size_t n) {
    std::memset(d, v, n);
    return hipSuccess;
}
template <typename T>
hipError_t hipGetSymbolAddress(void **p, T *symbol) {
    *p = (void *)symbol;
    return hipSuccess;
}
inline hipError_t hipGetDeviceCount(int *n) {
    *n = 1;
    return hipSuccess;
}
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    std::strcpy(p->gcnArchName, "gfx950");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
inline hipError_t hipDeviceSynchronize() { return fake::in_capture(true); }

inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = (hipStream_t)std::calloc(1, 8);
    return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
    std::free(s);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return fake::in_capture(false); }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    *g = (hipGraph_t)std::calloc(1, 8);
    return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, void *, char *, size_t) {
    *x = (hipGraphExec_t)std::calloc(1, 8);
    fake::graphs.fetch_add(1, std::memory_order_relaxed);
    return hipSuccess;
}
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipGraphDestroy(hipGraph_t g) {
    std::free(g);
    return hipSuccess;
}
inline hipError_t hipGraphExecDestroy(hipGraphExec_t g) {
    std::free(g);
    return hipSuccess;
}

inline hipError_t hipEventCreate(hipEvent_t *e) {
    *e = (hipEvent_t)std::calloc(1, 8);
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
inline hipError_t hipEventDestroy(hipEvent_t e) {
    std::free(e);
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
    *ms = 1.0f;
    return hipSuccess;
}
