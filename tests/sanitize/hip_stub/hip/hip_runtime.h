// The few HIP calls of the library's device-block pool, on host memory, so that
// the pool runs on the CPU under the host sanitizers.
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>

#define __host__
#define __device__

typedef enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 } hipError_t;
typedef struct stub_stream *hipStream_t;

extern size_t stub_capacity, stub_used, stub_calls;
extern thread_local int stub_device;

hipError_t hipMalloc(void **p, size_t bytes);
hipError_t hipFree(void *p);
inline hipError_t hipGetDevice(int *d) { *d = stub_device; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { stub_device = d; return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char *hipGetErrorString(hipError_t) { return "stub"; }
