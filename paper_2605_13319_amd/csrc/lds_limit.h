// Dynamic LDS of more than 64 KB has to be allowed per kernel, and on every device it runs on.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace pipesd {

// Allows `kernel` `bytes` of dynamic LDS on the current device, once: `done` (one word per kernel, static,
// zero at first) has a bit per device.  Devices beyond the 64th are asked every time.  Threads that come
// together may both ask; the bit is set only behind a call that succeeded.
inline hipError_t allow_lds(std::atomic<uint64_t>& done, const void* kernel, size_t bytes) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

}  // namespace pipesd
