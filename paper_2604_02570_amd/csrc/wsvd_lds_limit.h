// A kernel's limit of dynamic LDS above 64 KB is an attribute of the (kernel, device) pair: it is raised before the first launch
// on each device.  One object per kernel (a static of its launcher); concurrent callers may both raise it, to the same value.
#pragma once
#include <atomic>
#include <cstdint>

class LdsLimit {
  std::atomic<uint64_t> done_{0};                   // one bit per device; a device past the 64th raises it at every launch
 public:
  // `raise` sets the attribute on the current device, `device`; its status 0 is success
  template <class Raise>
  auto operator()(int device, Raise&& raise) -> decltype(raise()) {
    const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return decltype(raise())(0);
    const auto status = raise();
    if (status == decltype(raise())(0)) done_.fetch_or(bit, std::memory_order_release);
    return status;
  }
};
