// A device on the CPU for the host side of the library: memory is host memory,
// streams, events and graphs are nothing, launches are written down (launches.cpp).
#pragma once

#include "../../lanes/hip/hip_runtime.h"

#include <cstdlib>

#define __align__(n) __attribute__((aligned(n)))
enum { hipSuccess = 0, hipErrorNotInitialized = 3, hipErrorOutOfMemory = 2 };
enum { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2, hipStreamNonBlocking = 1, hipStreamCaptureModeThreadLocal = 1,
       hipDeviceAttributeWallClockRate = 1 };
struct ihipEvent_t;
struct ihipGraph;
struct hipGraphExec;
typedef ihipEvent_t *hipEvent_t;
typedef ihipGraph *hipGraph_t;
typedef hipGraphExec *hipGraphExec_t;
struct hipDeviceProp_t {
    size_t sharedMemPerBlock;
    int multiProcessorCount;
};
#define HIP_SYMBOL(x) x

inline size_t memory_left = (size_t)1 << 40;   // what hipMalloc has to give (bytes that are never touched cost nothing)

inline hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {
    p->sharedMemPerBlock = 160 << 10;
    p->multiProcessorCount = 256;
    return hipSuccess;
}
inline hipError_t hipDeviceGetAttribute(int *v, int, int) { return *v = 100000, hipSuccess; }
template <class T>
hipError_t hipMalloc(T **p, size_t bytes) {
    if (bytes > memory_left) return hipErrorOutOfMemory;
    return *p = (T *)std::malloc(bytes), *p ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipFree(void *p) { return std::free(p), hipSuccess; }
inline hipError_t hipMemcpy(void *to, const void *from, size_t n, int) { return std::memcpy(to, from, n), hipSuccess; }
inline hipError_t hipGetSymbolAddress(void **p, const void *symbol) { return *p = (void *)symbol, hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char *hipGetErrorString(hipError_t) { return "error"; }
inline hipError_t hipEventCreate(hipEvent_t *e) { return *e = nullptr, hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, int) { return *s = nullptr, hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamBeginCapture(hipStream_t, int) { return hipSuccess; }
inline hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { return *g = (hipGraph_t)std::malloc(1), hipSuccess; }
inline hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, void *, char *, size_t) {
    return *e = (hipGraphExec_t)std::malloc(1), hipSuccess;
}
inline hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipGraphDestroy(hipGraph_t g) { return std::free(g), hipSuccess; }
inline hipError_t hipGraphExecDestroy(hipGraphExec_t e) { return std::free(e), hipSuccess; }
