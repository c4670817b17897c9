// Raises a kernel's dynamic LDS limit to what a workgroup can have, once per kernel and device.
#pragma once
#include <atomic>
#include "common.h"

template <auto KERNEL>
bool grant_lds()
{
    static std::atomic<uint64_t> granted{0};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
    if (granted.load(std::memory_order_relaxed) >> dev & 1) return true;
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize,
                            144 * 1024) != hipSuccess)
        return false;
    granted.fetch_or(uint64_t(1) << dev, std::memory_order_relaxed);
    return true;
}
