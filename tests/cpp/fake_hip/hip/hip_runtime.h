// A HIP runtime of host memory and no device, for tests that compile the
// library's host code alone: one device of 256 CUs on which every call succeeds.
#pragma once

#include <stddef.h>
#include <stdint.h>

typedef int hipError_t;
enum : hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
typedef void *hipStream_t;
typedef void *hipGraph_t;
typedef void *hipGraphExec_t;
typedef void *hipGraphNode_t;
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount, hipDeviceAttributeMaxSharedMemoryPerBlock };

#define __host__
#define __device__

inline hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char *hipGetErrorName(hipError_t) { return "hipSuccess"; }
inline hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    return *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 163840, hipSuccess;
}
