// The limit of dynamic LDS of a kernel (64 KB unless asked for), set once on every device that launches it.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include <atomic>

namespace gsi {

// A static object per kernel.  A device that is through is remembered, a failure is not: the next call asks again.  Two
// threads that come first together both set the same value.
class LdsLimit {
 public:
  hipError_t allow(const void* kernel, int bytes) {
    int dev = 0;
    if (hipError_t e = hipGetDevice(&dev); e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? 1ull << dev : 0;
    if (done_.load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done_.fetch_or(bit, std::memory_order_relaxed);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace gsi
