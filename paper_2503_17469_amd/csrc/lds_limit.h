// Kernels with more than 64 KiB of dynamic LDS need their limit raised first: a host call per kernel and device, made once.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace omni {

constexpr size_t kLdsOfComputeUnit = 160 * 1024;

// One per kernel.  A kernel's limit is always the same number, the most that any of its launches asks for: host threads that
// step different networks (whose layers need different amounts) may be here at the same time, and a limit that followed the
// layers could be lowered by one between another's raising it and its launch.
class LdsLimit {
 public:
  void raise(const void* kernel, size_t bytes) {
    int device = 0;
    (void)hipGetDevice(&device);
    const uint64_t bit = device < 64 ? 1ull << device : 0;
    if (done_.load(std::memory_order_acquire) & bit) return;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess)
      done_.fetch_or(bit, std::memory_order_release);
  }

 private:
  std::atomic<uint64_t> done_{0};   // a bit per device
};

}  // namespace omni
