// Just enough of the HIP runtime, on host memory, to run the library's host
// entry points (tde_api.cpp) without a GPU: every call counts, and one call of
// a kind can be made to fail.
#pragma once
#include <cstdlib>
#include <cstring>

typedef int hipError_t;
constexpr int hipSuccess = 0, hipErrorOutOfMemory = 2;
typedef struct FakeStream* hipStream_t;
typedef struct FakeEvent* hipEvent_t;
typedef struct FakeGraph* hipGraph_t;
typedef struct FakeExec* hipGraphExec_t;
enum { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipStreamCaptureModeThreadLocal = 1 };

namespace fake {
inline int fail_malloc = -1;  // the malloc that fails, counted from now; -1: none
inline int fail_async = -1;   // the same for asynchronous copies
inline int syncs = 0, pending = 0;  // stream waits; asynchronous steps not yet waited for
inline int countdown(int* k) { return *k >= 0 && (*k)-- == 0; }
}  // namespace fake

inline hipError_t hipMalloc(void** p, size_t n) {
    if (fake::countdown(&fake::fail_malloc)) return hipErrorOutOfMemory;
    return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory;
}
template <class T>
hipError_t hipMalloc(T** p, size_t n) {
    return hipMalloc((void**)p, n);
}
inline hipError_t hipFree(void* p) {
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, int) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int, hipStream_t) {
    if (fake::countdown(&fake::fail_async)) return hipErrorOutOfMemory;
    std::memcpy(d, s, n);
    ++fake::pending;
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) {
    ++fake::syncs;
    fake::pending = 0;
    return hipSuccess;
}
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = nullptr;
    return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t, int) { return hipSuccess; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    *g = (hipGraph_t)1;
    return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, void*, char*, size_t) {
    *e = (hipGraphExec_t)1;
    return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = (hipEvent_t)1;
    return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
