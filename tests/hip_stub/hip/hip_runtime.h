// A stand-in for the HIP runtime that lets the HOST side of the library (configuration checks, arena layout,
// per-cache bookkeeping, export / import packing) be compiled for the CPU and run under AddressSanitizer and
// UndefinedBehaviorSanitizer.  "Device" memory is host memory, streams and events are dummies, nothing is launched
// (the kernel launchers are replaced by no-ops in launch_stubs.cpp).  Test infrastructure only.
#pragma once
#include <cstdint>
#include <cstdlib>
#include <cstring>

#define __host__
#define __device__
#define __global__
#define __forceinline__ inline __attribute__((always_inline))
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) x

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidDevice = 101 };
typedef struct hipStubStream* hipStream_t;
typedef struct hipStubEvent* hipEvent_t;
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount = 1 };

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

inline hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
inline hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return "stub"; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline int stub_cus = 256;             // compute units of the pretended device
inline bool stub_mean_in_score;        // last scoring launch: whether its blocks form the row mean
// last attention launch: key ranges, scoring blocks per cache inside it; last step: whether the rewrite takes the merge along and
// scoring selects
inline int stub_splits, stub_side_blocks, stub_merge, stub_score_selects;
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = stub_cus; return hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
inline hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline int stub_stream_waits = 0;      // waits enqueued so far: a step on two streams makes two, one in order none
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { ++stub_stream_waits; return hipSuccess; }
inline hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
inline hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
template <typename T>
inline hipError_t hipGetSymbolAddress(void** p, T& sym) { *p = (void*)&sym; return hipSuccess; }
