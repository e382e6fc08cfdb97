// Host-side helpers of the kernel launchers.
#ifndef CHUNKFT_LAUNCH_H
#define CHUNKFT_LAUNCH_H

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "internal.h"

namespace chunkft {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Allows `Kern` to ask for `bytes` of dynamic LDS on the current device.  The limit is a per-device
// attribute of the kernel; raising it is idempotent, so a race between threads only repeats the call.
template <auto Kern>
int raise_lds_limit(size_t bytes) {
  static std::atomic<bool> done[kMaxDevices] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return (int)hipErrorInvalidDevice;
  const bool known = dev >= 0 && dev < kMaxDevices;
  if (known && done[dev].load(std::memory_order_acquire)) return 0;
  const hipError_t e = hipFuncSetAttribute((const void*)Kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e != hipSuccess) return (int)e;
  if (known) done[dev].store(true, std::memory_order_release);
  return 0;
}

}  // namespace chunkft
#endif
