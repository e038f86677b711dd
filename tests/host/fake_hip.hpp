// A stand-in for the HIP runtime, linked into a host test program: the library's
// own calls of these functions land here.  Device memory is host memory, copies
// and clears happen at once, kernels do nothing, and an allocation can be made
// to fail.  Every copy and clear checks that its device side lies in live
// memory.
#pragma once
#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>

namespace fake {
inline std::mutex mtx;
inline std::map<char *, size_t> live;
inline size_t bytes = 0;          // live device bytes
inline long mallocs = 0, launches = 0;
inline long fail_in = -1;         // the allocation that fails, counted down; < 0: none
inline long stale = 0;            // copies and clears outside live memory
inline long frees = 0;            // of device memory: each waits for the whole device
inline std::atomic<int> slow_frees{0};   // so many frees take a second
inline bool ended = false;        // the runtime is gone
inline long late = 0;             // calls after that
inline bool is_live(const void *p, size_t n) {
  auto it = live.upper_bound((char *)p);
  if (it == live.begin()) return false;
  --it;
  return (char *)p + n <= it->first + it->second;
}
inline void touch(const void *p, size_t n) {
  std::lock_guard<std::mutex> l(mtx);
  if (!is_live(p, n)) ++stale;
}
}  // namespace fake

extern "C" {
hipError_t hipInit(unsigned) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 1, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "fake"; }
hipError_t hipMalloc(void **p, size_t n) {
  std::lock_guard<std::mutex> l(fake::mtx);
  if (fake::fail_in == 0) return hipErrorOutOfMemory;   // stays: the library tries once more
  if (fake::fail_in > 0) --fake::fail_in;
  char *q = (char *)std::malloc(n);
  if (!q) return hipErrorOutOfMemory;
  ++fake::mallocs;
  fake::live[q] = n;
  fake::bytes += n;
  *p = q;
  return hipSuccess;
}
hipError_t hipFree(void *p) {
  if (fake::slow_frees > 0 && fake::slow_frees-- > 0) std::this_thread::sleep_for(std::chrono::seconds(1));
  std::lock_guard<std::mutex> l(fake::mtx);
  if (fake::ended) ++fake::late;
  auto it = fake::live.find((char *)p);
  if (it == fake::live.end()) return hipErrorInvalidValue;
  ++fake::frees;
  fake::bytes -= it->second;
  fake::live.erase(it);
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return *p = std::malloc(n), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) {
  if (k == hipMemcpyHostToDevice || k == hipMemcpyDeviceToDevice) fake::touch(d, n);
  if (k == hipMemcpyDeviceToHost || k == hipMemcpyDeviceToDevice) fake::touch(s, n);
  if (!fake::stale) std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) {
  fake::touch(d, n);
  if (!fake::stale) std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)0x10, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *c) { return *c = hipStreamCaptureStatusNone, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = (hipEvent_t)0x20, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)0x20, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 0.0f, hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { return *n = 1, hipSuccess; }
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return ++fake::launches, hipSuccess; }
hipError_t hipLaunchCooperativeKernel(const void *, dim3, dim3, void **, unsigned, hipStream_t) {
  return ++fake::launches, hipSuccess;
}
static dim3 call_grid, call_block;
static size_t call_lds;
static hipStream_t call_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t l, hipStream_t s) {
  return call_grid = g, call_block = b, call_lds = l, call_stream = s, hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *l, hipStream_t *s) {
  return *g = call_grid, *b = call_block, *l = call_lds, *s = call_stream, hipSuccess;
}
void **__hipRegisterFatBinary(const void *) {
  static void *handle;
  return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
}
