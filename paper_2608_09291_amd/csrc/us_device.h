// Compute units of the current device, shared by the host sides.
#ifndef UNIONSPARSE_US_DEVICE_H
#define UNIONSPARSE_US_DEVICE_H

#include <hip/hip_runtime.h>

#include <atomic>

namespace us_device {

inline int compute_units_of(int dev) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    return n;
}

// 256 (an MI355X) when no device answers. Every call plans with it: where all
// visible devices have the same number, as on any one node, it is queried once
// and the current device is not asked for (53 ns of a 3 us launch).
inline int compute_units() {
    static std::atomic<int> common{0};                     // 0: not known yet, -1: they differ
    int c = common.load(std::memory_order_relaxed);
    if (c > 0) return c;
    int dev = 0;
    if (c == 0) {
        int count = 0;
        if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) return 256;
        c = compute_units_of(0);
        for (int d = 1; d < count; ++d)
            if (compute_units_of(d) != c) c = -1;
        common.store(c, std::memory_order_relaxed);
        if (c > 0) return c;
    }
    return hipGetDevice(&dev) == hipSuccess ? compute_units_of(dev) : 256;
}

}  // namespace us_device

#endif  // UNIONSPARSE_US_DEVICE_H
