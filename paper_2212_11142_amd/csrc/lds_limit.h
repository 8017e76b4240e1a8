// The dynamic LDS limit of a kernel (above 64 KB it has to be raised), set once per device.
#pragma once
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdint>

namespace bgp {

// One static object per kernel. The attribute belongs to the current device's copy of the
// kernel, so each device sets its own; a call that failed is made again. Safe with several
// threads: two that come first together both set it.
class LdsLimit {
  std::atomic<uint64_t> done_{0};  // bit d: set on device d

 public:
  hipError_t set(const void *kernel, int bytes) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;  // (past 64: every time)
    if (done_.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }
};

}  // namespace bgp
