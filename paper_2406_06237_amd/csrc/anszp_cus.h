// Host state shared by the library's sources (internal to the library).
//
// Compute units of a device: queried once per device; the cache is a
// table of atomics, so concurrent callers at worst both query.
#ifndef ANSZP_CUS_H
#define ANSZP_CUS_H

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

inline uint32_t device_cus(int dev) {
    static std::atomic<uint32_t> cached[64];
    if (dev < 0 || dev >= 64) return 256u;
    uint32_t n = cached[dev].load(std::memory_order_relaxed);
    if (!n) {
        int count = 0;
        if (hipDeviceGetAttribute(&count, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || count <= 0) count = 256;
        n = static_cast<uint32_t>(count);
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

// of the current device
inline uint32_t device_cus() {
    int dev = 0;
    return hipGetDevice(&dev) == hipSuccess ? device_cus(dev) : 256u;
}

// The bound of every wait between wavefronts or workgroups, in polls and one more; 0: each kernel's own.  Tests lower
// it (anszp_test_set_spin_limit) to see what a wait that is given up leads to.
inline std::atomic<uint32_t>& spin_limit_for_tests() {
    static std::atomic<uint32_t> polls{0};
    return polls;
}

#endif
