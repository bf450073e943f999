// Host stand-in for the part of the HIP runtime and language that the library's
// launch code and windowed-lane kernels use: one thread per work item, LDS as a
// global array, barriers as pthread barriers (tests/windowed_host.cpp).
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>

#define __device__
#define __global__
#define __host__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
extern thread_local dim3 threadIdx, blockIdx, blockDim, gridDim;
void host_block_barrier();
void host_wave_barrier();
inline void __syncthreads() { host_block_barrier(); }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
#define __builtin_amdgcn_fence(order, scope)
#define __builtin_amdgcn_wave_barrier host_wave_barrier
#define __builtin_amdgcn_sched_barrier(mask)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __all(x) (x)
template <typename A>
A atomicAdd(A *p, A v) { return __sync_fetch_and_add(p, v); }
template <typename A, typename B>
A atomicExch(A *p, B v) { return __sync_lock_test_and_set(p, (A)v); }
inline void __threadfence() {}

typedef int hipError_t;
typedef void *hipStream_t;
typedef void *hipEvent_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone };
enum hipStreamCaptureMode { hipStreamCaptureModeRelaxed };
enum {
  hipDeviceAttributeMaxSharedMemoryPerBlock,
  hipDeviceAttributeNumberOfXccs,
  hipDeviceAttributeMultiprocessorCount,
  hipEventDisableTiming,
  hipHostMallocDefault,
  hipMemcpyHostToDevice
};
inline hipError_t hipGetDevice(int *d) { return *d = 0; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int *v, int a, int) {
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 163840 : (a == hipDeviceAttributeNumberOfXccs ? 8 : 1);
  return hipSuccess;
}
inline const char *hipGetErrorString(hipError_t) { return "host"; }
template <typename T>
hipError_t hipMalloc(T **p, size_t n) {
  *p = static_cast<T *>(aligned_alloc(256, (n + 255) / 256 * 256));
  return hipSuccess;
}
inline hipError_t hipFree(void *p) { return free(p), hipSuccess; }
inline hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return hipMalloc(p, n); }
inline hipError_t hipFreeAsync(void *p, hipStream_t) { return hipFree(p); }
template <typename T>
hipError_t hipHostMalloc(T **p, size_t n, int) { return hipMalloc(p, n); }
inline hipError_t hipHostFree(void *p) { return hipFree(p); }
inline hipError_t hipMemcpy(void *d, const void *s, size_t n, int) { return memcpy(d, s, n), hipSuccess; }
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, int, hipStream_t) { return memcpy(d, s, n), hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { return hipSuccess; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
  *s = hipStreamCaptureStatusNone;
  return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, int) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, int) { return *e = e, hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
inline hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  return *n = 1, hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t);
