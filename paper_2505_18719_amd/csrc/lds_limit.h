// Dynamic LDS above 64 KB has to be allowed for a kernel on each device that it is launched on.
#pragma once

#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstddef>
#include <cstdint>

namespace vla {

// One per kernel (a static of its launcher), which always asks for the same size.  The attribute is set once per device;
// several threads may ask at once, and a call that failed is made again.
class LdsLimit {
 public:
  hipError_t allow(const void* kernel, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;  // further devices: set at each launch
    if (done_.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace vla
