// Host stand-in for the HIP runtime calls of the call-by-call heaps, so that
// the library's own host code runs on the CPU: device memory is host memory,
// and a launch runs the kernel as an emulated wave before it returns.  Test
// infrastructure only.
#pragma once
#include <cstdlib>
#include <cstring>
#include <functional>

#include "../../hip/hip_runtime.h"

#define __global__

typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2 };
typedef void* hipStream_t;
typedef int hipMemcpyKind;
enum { hipMemcpyHostToDevice, hipMemcpyDeviceToHost };
enum { hipStreamNonBlocking = 1, hipHostMallocCoherent = 1, hipHostMallocMapped = 2,
       hipHostMallocPortable = 4 };
struct dim3 {
  unsigned x;
  dim3(unsigned n) : x(n) {}
};

#define __HIP_MEMORY_SCOPE_SYSTEM 0
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)

// Run f as a wave of 64 lanes (emu_host.cpp).
void emu_run_wave(const std::function<void()>& f);
// Called for every hipHostFree, before the memory goes.
extern void (*emu_on_host_free)();
extern int emu_host_pages;  // hipHostMalloc'd and not freed yet

#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
  emu_run_wave([=] { kernel(__VA_ARGS__); })

inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  static int one;
  return *s = &one, hipSuccess;
}
extern int emu_stream_waits;  // hipStreamSynchronize calls
inline hipError_t hipStreamSynchronize(hipStream_t) {
  __atomic_fetch_add(&emu_stream_waits, 1, __ATOMIC_RELAXED);
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  return std::memcpy(d, s, n), hipSuccess;
}
inline hipError_t hipMalloc(void** p, size_t n) {
  return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipFree(void* p) { return std::free(p), hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  __atomic_fetch_add(&emu_host_pages, 1, __ATOMIC_RELAXED);
  return (*p = std::aligned_alloc(4096, n)) ? hipSuccess : hipErrorOutOfMemory;
}
inline hipError_t hipHostFree(void* p) {
  if (emu_on_host_free) emu_on_host_free();
  __atomic_fetch_sub(&emu_host_pages, 1, __ATOMIC_RELAXED);
  return std::free(p), hipSuccess;
}
inline hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  return *d = h, hipSuccess;
}
