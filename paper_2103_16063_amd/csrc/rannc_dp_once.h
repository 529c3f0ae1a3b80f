// Something a process has to ask of the runtime once for every device it uses.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

namespace rannc {

// done: a bit per device.  ask() runs for the current device unless it has succeeded there before; a
// failure is reported and not kept, so that a later call asks again.  (Two threads may both ask.)
template <typename CurrentDevice, typename Ask>
hipError_t once_per_device(std::atomic<uint64_t> &done, CurrentDevice current, Ask ask) {
  int dev = -1;
  const hipError_t e = current(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;  // (beyond 64 devices every call asks)
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  const hipError_t r = ask();
  if (r == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return r;
}

// A kernel whose LDS, its own and the dynamic part, can exceed the default 64 KiB: the limit belongs to its function on one device.
// (Asked for whatever a launch needs: how much a kernel has of its own changes with its code.)
inline hipError_t allow_lds(std::atomic<uint64_t> &done, const void *kernel, int bytes) {
  return once_per_device(done, [](int *dev) { return hipGetDevice(dev); }, [&] {
    return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  });
}

}  // namespace rannc
