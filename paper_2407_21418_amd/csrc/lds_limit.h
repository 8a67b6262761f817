// A kernel gets more than 64 KB of dynamic LDS only if its limit was raised on the device it is launched on.
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>

namespace ftk {

// Raises KERNEL's limit to a CU's whole LDS, once on each device it is launched on (the attribute is kept per device).
template <auto KERNEL> hipError_t raise_lds_limit() {
    static std::mutex mu;
    static bool done[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!done[dev]) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, 163840);
        if (e != hipSuccess) return e;
        done[dev] = true;
    }
    return hipSuccess;
}

}  // namespace ftk
