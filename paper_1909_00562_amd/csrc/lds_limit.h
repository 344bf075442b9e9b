// Kernels with more dynamic LDS than a launch gets unasked.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

namespace asx {

// Devices on which a kernel's limit has been raised, one object per kernel.  The limit belongs to the kernel as loaded on a
// device, so each device of the process needs its own call; setting it twice is harmless, so threads need no lock.
class LdsLimit {
 public:
  hipError_t raise(const void* kernel, int bytes) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev >= 0 && dev < 64 ? uint64_t(1) << dev : 0;   // past 64 devices: on every launch
    if (done_.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess) done_.fetch_or(bit, std::memory_order_release);
    return e;
  }

 private:
  std::atomic<uint64_t> done_{0};
};

}  // namespace asx
