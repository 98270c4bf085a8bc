// The few HIP names that the library's memory pool uses, over a device memory of
// `budget` bytes on the host (pool_check.cpp).
#pragma once
#include <cstddef>
#include <cstdlib>
#include <map>

typedef enum {
  hipSuccess = 0,
  hipErrorOutOfMemory = 2,
  hipErrorInvalidDevice = 101,
  hipErrorStreamCaptureUnsupported = 900
} hipError_t;
typedef void* hipStream_t;
typedef enum { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice } hipMemcpyKind;
enum { hipStreamNonBlocking = 1 };

namespace stub {
inline size_t budget = size_t(1) << 40, used = 0;
inline bool may_wait = true;   // false: as in a thread that is capturing
inline std::map<void*, size_t> live;
}  // namespace stub

inline hipError_t hipMalloc(void** p, size_t bytes) {
  *p = nullptr;
  if (stub::used + bytes > stub::budget) return hipErrorOutOfMemory;
  *p = std::malloc(1);
  stub::live[*p] = bytes;
  stub::used += bytes;
  return hipSuccess;
}
inline hipError_t hipFree(void* p) {
  if (!stub::may_wait) return hipErrorStreamCaptureUnsupported;
  if (!p) return hipSuccess;
  stub::used -= stub::live.at(p);
  stub::live.erase(p);
  std::free(p);
  return hipSuccess;
}
inline hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = nullptr;
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
