// The limit of dynamic LDS that a kernel starts with, raised where a launch needs more.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace bmx {

// Lets `kern` have all of a CU's LDS (160 KB) as dynamic LDS where `bytes` is more than the default limit; asked for
// once per device, by the caller's array of one flag each.  Threads may meet here: they ask for the same thing.
static inline hipError_t allow_lds(const void* kern, size_t bytes, std::atomic<bool> (&asked)[64]) {
  if (bytes <= 64 * 1024) return hipSuccess;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (asked[dev].load(std::memory_order_acquire)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess) asked[dev].store(true, std::memory_order_release);
  return e;
}

}  // namespace bmx
