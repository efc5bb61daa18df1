// lds_limit.h -- dynamic LDS above 64 KB for a kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace pd {

// Lets `kernel` run with `bytes` of dynamic LDS on the current device.  The
// attribute belongs to one device's copy of the kernel, so it is set once per
// device (bits of `done`, the kernel's own; past 64 devices on every call).
inline hipError_t allow_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = (unsigned)dev < 64 ? 1ull << dev : 0ull;
  if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

}  // namespace pd
