// The dynamic-LDS limit of a kernel (host side).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

namespace rbgs {

// Lets a kernel take up to `bytes` of dynamic LDS, once per device (`done`: a
// bit per device, of the caller's static).  The limit belongs to the kernel, not
// to a launch: set to each launch's own need, a small launch on one thread
// could lower it between another thread's setting and launch.
inline hipError_t allow_dynamic_lds(const void* kernel, size_t bytes, std::atomic<uint64_t>& done) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? uint64_t(1) << dev : 0;
    if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes));
    if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
    return e;
}

}  // namespace rbgs
