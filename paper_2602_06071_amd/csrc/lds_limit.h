// Work-groups with more LDS than a kernel gets by default.
#pragma once
#include <hip/hip_runtime.h>

#include <atomic>

namespace fs {

constexpr size_t kLdsDefault = 64 * 1024, kLdsMost = 160 * 1024;  // a kernel's default limit, a CU's LDS

// The current device, without asking where the process sees only one (a few hundredths of a microsecond
// per launch).
inline hipError_t current_device(int* dev) {
  static const int count = [] {
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess) { (void)hipGetLastError(); n = 0; }
    return n;
  }();
  *dev = 0;
  return count == 1 ? hipSuccess : hipGetDevice(dev);
}

// Raises the dynamic-LDS limit of `kernel` on the current device if a launch with `lds` bytes needs it:
// the limit belongs to a (kernel, device) pair, so each device is noted in a mask of its own per
// kernel (a template argument, hence one mask each).  Threads may race here: at worst the limit is set twice.
template <auto kernel>
hipError_t allow_lds(size_t lds) {
  if (lds <= kLdsDefault) return hipSuccess;
  static std::atomic<uint64_t> raised{0};
  int dev = 0;
  hipError_t e = current_device(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = dev >= 0 && dev < 64 ? (uint64_t)1 << dev : 0;  // (further devices: set on every launch)
  if (raised.load(std::memory_order_relaxed) & bit) return hipSuccess;
  e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMost);
  if (e == hipSuccess) raised.fetch_or(bit, std::memory_order_relaxed);
  return e;
}

}  // namespace fs
