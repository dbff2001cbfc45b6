// A HIP runtime of host memory and no device, for tests that compile the
// library's host code alone: one device of 256 CUs.  Streams, events and graphs
// are defined by the test that uses them.
#pragma once

#include <stddef.h>
#include <stdint.h>

typedef int hipError_t;
enum : hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
typedef void *hipStream_t;
typedef void *hipEvent_t;
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

enum : unsigned { hipHostMallocCoherent = 0x40000000, hipEventDisableTiming = 2, hipStreamNonBlocking = 1 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal = 1 };

hipError_t hipMalloc(void **p, size_t bytes);
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned flags);
hipError_t hipHostGetDevicePointer(void **dev, void *host, unsigned flags);
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned flags);
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st);
hipError_t hipEventSynchronize(hipEvent_t e);
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned flags);
hipError_t hipStreamSynchronize(hipStream_t st);
hipError_t hipStreamCreateWithFlags(hipStream_t *st, unsigned flags);
hipError_t hipStreamDestroy(hipStream_t st);
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus *s);
hipError_t hipStreamBeginCapture(hipStream_t st, hipStreamCaptureMode m);
hipError_t hipStreamEndCapture(hipStream_t st, hipGraph_t *g);
hipError_t hipGraphGetRootNodes(hipGraph_t g, hipGraphNode_t *nodes, size_t *n);
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *node, char *log, size_t bytes);
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st);
hipError_t hipGraphExecDestroy(hipGraphExec_t x);
hipError_t hipGraphDestroy(hipGraph_t g);
