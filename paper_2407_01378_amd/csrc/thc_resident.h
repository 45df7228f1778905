// What the current device keeps resident of a kernel: the size of a persistent grid.
//
// The queries take tens of microseconds, more than a small call, so their answers are kept: per
// device, and per kernel by the shape of its workgroup (threads and dynamic LDS both decide how many
// fit a CU).  The tables have a fixed size and no lock; a thread that finds another's half-filled
// table asks the device once more.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>

namespace thc {

inline int current_device() {
    int dev = -1;
    return hipGetDevice(&dev) == hipSuccess ? dev : -1;
}

// Compute units of the current device, 0 if it does not say.
inline int device_cus() {
    constexpr int kDevices = 64;
    static std::atomic<int> known[kDevices];
    const int dev = current_device();
    if (dev < 0) return 0;
    int cus = dev < kDevices ? known[dev].load(std::memory_order_relaxed) : 0;
    if (cus == 0) {
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 0) return 0;
        if (dev < kDevices) known[dev].store(cus, std::memory_order_relaxed);
    }
    return cus;
}

// Workgroups of `threads` threads and `lds` bytes of dynamic LDS that the current device keeps
// resident at once, 0 if it does not say.
template <auto kernel>
uint32_t resident_grid(uint32_t threads, uint32_t lds = 0) {
    constexpr uint32_t kShapes = 32;
    static std::atomic<uint64_t> known[kShapes];   // (device + 1, waves, LDS words) << 32 | workgroups; 0: free
    const int dev = current_device();
    if (dev < 0) return 0;
    const uint64_t shape = ((uint64_t)(dev + 1) << 22 | (uint64_t)(threads / 64u) << 17 | lds / 4u) & 0xFFFFFFFFu;
    uint32_t at = 0;
    for (; at < kShapes; ++at) {
        const uint64_t k = known[at].load(std::memory_order_relaxed);
        if (k >> 32 == shape) return (uint32_t)k;
        if (k == 0) break;
    }
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, (int)threads, lds) != hipSuccess || occ < 1) return 0;
    const uint32_t grid = (uint32_t)(occ * device_cus());
    if (grid != 0) known[at < kShapes ? at : shape % kShapes].store(shape << 32 | grid, std::memory_order_relaxed);
    return grid;
}

// Lets the kernel be launched with `lds` bytes of dynamic LDS on the current device, which beyond 64 KB
// it has to be told once.
template <auto kernel>
bool allow_lds(uint32_t lds) {
    if (lds <= 65536u) return true;
    static std::atomic<uint64_t> told;   // a bit per device
    const int dev = current_device();
    if (dev < 0) return false;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0u;
    if (told.load(std::memory_order_relaxed) & bit) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 163840) !=
        hipSuccess)
        return false;
    told.fetch_or(bit, std::memory_order_relaxed);
    return true;
}

}  // namespace thc
