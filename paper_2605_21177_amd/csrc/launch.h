// Host-side helpers of the kernel launchers.
#ifndef CHUNKFT_LAUNCH_H
#define CHUNKFT_LAUNCH_H

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "internal.h"

namespace chunkft {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Runs a call in pieces of at most `most` elements (0: it cannot run): run(p, s) with the range of a piece and the sinks moved to
// its first element.
template <class Run>
int in_pieces(const WgradProblem& p, const Sinks& s, int64_t most, Run&& run) {
  if (most <= 0) return (int)hipErrorInvalidValue;
  for (int64_t b = p.begin; b < p.end;) {
    WgradProblem q = p;
    Sinks t = s;
    q.begin = b;
    q.end = p.end - b > most ? b + most : p.end;
    const int64_t at = b - p.begin;
    if (s.g) t.g += at;
    if (s.ws) t.ws += at;
    if (s.master) { t.master += at; t.m += at; t.v += at; }
    const int err = run(q, t);
    if (err != 0) return err;
    b = q.end;
  }
  return 0;
}

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
