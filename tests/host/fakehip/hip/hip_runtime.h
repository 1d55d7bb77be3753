// The HIP calls that csrc/workspace.cpp makes, for workspace_checks.cpp, which
// defines them: a test double of the runtime, no device behind it.
#pragma once

#include <cstddef>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorStreamCaptureUnsupported = 900 };
enum hipStreamCaptureMode {
    hipStreamCaptureModeGlobal = 0,
    hipStreamCaptureModeThreadLocal,
    hipStreamCaptureModeRelaxed
};
using hipStream_t = struct FakeStream *;
constexpr unsigned hipHostMallocMapped = 2;
constexpr unsigned hipHostMallocCoherent = 0x40000000;
constexpr unsigned hipStreamNonBlocking = 1;

hipError_t hipGetLastError();
hipError_t hipGetDevice(int *);
hipError_t hipSetDevice(int);
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *);
hipError_t hipMalloc(void **, size_t);
hipError_t hipFree(void *);
hipError_t hipMallocAsync(void **, size_t, hipStream_t);
hipError_t hipFreeAsync(void *, hipStream_t);
hipError_t hipHostMalloc(void **, size_t, unsigned);
hipError_t hipHostFree(void *);
hipError_t hipHostGetDevicePointer(void **, void *, unsigned);
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned);
hipError_t hipStreamDestroy(hipStream_t);
hipError_t hipStreamSynchronize(hipStream_t);
