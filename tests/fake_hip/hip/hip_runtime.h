// The few HIP calls that slot_pool.h makes, for tests of it without a GPU: streams are numbers, and the test says which GPU
// each belongs to, which GPU is current and which streams are capturing.
#pragma once
#include <stddef.h>
#include <stdlib.h>

#include <map>
#include <set>

enum hipError_t { hipSuccess = 0, hipErrorInvalidHandle = 400, hipErrorStreamCaptureImplicit = 906 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
typedef struct ihipStream_t* hipStream_t;
typedef int hipDevice_t;
#define hipStreamLegacy ((hipStream_t)1)
#define hipStreamPerThread ((hipStream_t)2)
constexpr unsigned hipHostMallocDefault = 0, hipHostMallocPortable = 1;

namespace fake_hip {
inline int current = 0;
inline std::map<hipStream_t, int> device;                    // of the streams that exist, but for the null streams
inline std::set<hipStream_t> capturing;
inline hipError_t last = hipSuccess;
inline hipError_t is(hipError_t e) { return e == hipSuccess ? e : last = e; }
inline bool null(hipStream_t s) { return s == nullptr || s == hipStreamLegacy; }
}  // namespace fake_hip

inline hipError_t hipGetDevice(int* d) { *d = fake_hip::current; return hipSuccess; }
inline hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d)
{
    if (fake_hip::null(s)) return hipGetDevice(d);
    const auto it = fake_hip::device.find(s);
    if (it == fake_hip::device.end()) return fake_hip::is(hipErrorInvalidHandle);
    *d = it->second;
    return hipSuccess;
}
inline hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* status)
{
    if (fake_hip::null(s) && !fake_hip::capturing.empty()) return fake_hip::is(hipErrorStreamCaptureImplicit);
    *status = fake_hip::capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned = 0) { *p = malloc(n); return hipSuccess; }
inline hipError_t hipGetLastError() { const hipError_t e = fake_hip::last; fake_hip::last = hipSuccess; return e; }
inline hipError_t hipPeekAtLastError() { return fake_hip::last; }
