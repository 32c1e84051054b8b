// Compute units of the current device (host code, internal to the library): queried once per device; the cache is a
// table of atomics, so concurrent callers at worst both query.
#ifndef ANSZP_CUS_H
#define ANSZP_CUS_H

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

inline uint32_t device_cus() {
    static std::atomic<uint32_t> cached[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256u;
    uint32_t n = cached[dev].load(std::memory_order_relaxed);
    if (!n) {
        int count = 0;
        if (hipDeviceGetAttribute(&count, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || count <= 0) count = 256;
        n = static_cast<uint32_t>(count);
        cached[dev].store(n, std::memory_order_relaxed);
    }
    return n;
}

#endif
