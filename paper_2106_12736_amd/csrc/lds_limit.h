// The dynamic LDS limit of a kernel belongs to the device it is set on.
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace fdc {

// Raise a kernel's dynamic LDS limit to `bytes` on the current device: at its first launch
// there (a failure is tried again at the next).
template <auto Kern>
hipError_t allow_lds(size_t bytes) {
  static std::atomic<std::uint64_t> raised{0};  // a bit a device
  int dev = 0;
  if (hipError_t e = hipGetDevice(&dev)) return e;
  const std::uint64_t bit = dev >= 0 && dev < 64 ? std::uint64_t(1) << dev : 0;
  if (raised.load(std::memory_order_relaxed) & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(Kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) raised.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

}  // namespace fdc
