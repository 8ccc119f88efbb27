// Compute units of the current device, shared by the host sides.
#ifndef UNIONSPARSE_US_DEVICE_H
#define UNIONSPARSE_US_DEVICE_H

#include <hip/hip_runtime.h>

#include <atomic>

namespace us_device {

// Queried once per device; 256 (an MI355X) when no device answers.
inline int compute_units() {
    static std::atomic<int> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n <= 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

}  // namespace us_device

#endif  // UNIONSPARSE_US_DEVICE_H
