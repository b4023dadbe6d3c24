// Decisions of the host code that need no device, free of HIP so that they
// can be checked without one.
#pragma once

#include <cstddef>
#include <cstdint>

namespace sdprt {

// Blocks of `threads` threads that one launch may have: the runtime refuses
// 2^32 threads or more in a dimension.
constexpr int64_t launch_blocks(int threads) { return (int64_t)0xffffffff / threads; }

// How many of `n` segments one launch takes: at most max_segs, and only so many
// that their blocks (blocks_of(k)) together stay within max_blocks; the first in
// any case.
template <class BlocksOf>
int segments_that_fit(int n, int max_segs, int64_t max_blocks, BlocksOf blocks_of) {
    int k = 0;
    int64_t blocks = 0;
    for (; k < n && k < max_segs; ++k) {
        const int64_t b = blocks_of(k);
        if (k > 0 && b > max_blocks - blocks) break;
        blocks += b;
    }
    return k;
}

// An allocation as the device addresses it.
struct Allocation {
    const char *base;
    size_t bytes;
};

// The device's address of pinned host memory [p, p + bytes), for kernels that
// work on it in place: only if it is 16-byte aligned and the whole range lies in
// one allocation.  (The two ends alone do not say so: between two pinned blocks
// may lie memory that the device cannot reach, and a kernel's access there
// faults, where a copy by the runtime does not.)
// device_address(p): the device's address of host address p, or NULL;
// allocation_of(d, &a): the allocation around device address d, or false.
template <class DeviceAddress, class AllocationOf>
bool map_range(const void *p, size_t bytes, DeviceAddress device_address, AllocationOf allocation_of, void **out) {
    void *d = device_address(p);
    if (!d || (uintptr_t)d % 16 != 0) return false;
    Allocation a{};
    if (!allocation_of(d, &a) || (const char *)d < a.base) return false;
    const size_t before = (size_t)((const char *)d - a.base);
    if (before > a.bytes || bytes > a.bytes - before) return false;
    *out = d;
    return true;
}

}  // namespace sdprt
