// Compute units of the current device.  Internal to the library.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>

namespace lbm {

// Asked once per device; 256 if the runtime cannot say.
inline int compute_units() {
    static std::atomic<int> known[64];
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    cus = known[dev].load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        return 256;
    known[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

}  // namespace lbm
