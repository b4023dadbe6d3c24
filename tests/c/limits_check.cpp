// Checks sdp_limits.h without a device; prints "ok" or exits 1.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "sdp_limits.h"

using namespace sdprt;

#define CHECK(x)                                                       \
    do {                                                               \
        if (!(x)) {                                                    \
            std::printf("line %d: %s\n", __LINE__, #x);                \
            std::exit(1);                                              \
        }                                                              \
    } while (0)

static char *at(uintptr_t x) { return (char *)x; }

// Host memory of three pinned blocks: [0x10000, 0x20000) and, after a hole,
// [0x30000, 0x40000) and right behind it [0x40000, 0x50000); the device has
// each at the same address plus `shift`.
static void check_map(uintptr_t shift) {
    struct Block {
        uintptr_t base;
        size_t bytes;
    };
    static const Block blocks[3] = {{0x10000, 0x10000}, {0x30000, 0x10000}, {0x40000, 0x10000}};
    auto device_address = [&](const void *p) -> void * {
        for (const Block &b : blocks)
            if ((uintptr_t)p >= b.base && (uintptr_t)p < b.base + b.bytes) return at((uintptr_t)p + shift);
        return nullptr;
    };
    auto allocation_of = [&](const void *d, Allocation *a) {
        for (const Block &b : blocks)
            if ((uintptr_t)d - shift >= b.base && (uintptr_t)d - shift < b.base + b.bytes) {
                *a = {at(b.base + shift), b.bytes};
                return true;
            }
        return false;
    };
    auto mapped = [&](uintptr_t p, size_t bytes) -> uintptr_t {
        void *out = nullptr;
        return map_range(at(p), bytes, device_address, allocation_of, &out) ? (uintptr_t)out : 0;
    };
    CHECK(mapped(0x10000, 0x10000) == 0x10000 + shift);
    CHECK(mapped(0x10010, 0xfff0) == 0x10010 + shift);
    CHECK(mapped(0x1fff0, 16) == 0x1fff0 + shift);
    CHECK(mapped(0x10000, 0x10001) == 0);  // one byte over
    CHECK(mapped(0x1fff0, 17) == 0);
    CHECK(mapped(0x10000, 0x30000) == 0);  // both ends pinned, a hole between
    CHECK(mapped(0x3fff0, 32) == 0);       // two allocations, no hole: copies as well
    CHECK(mapped(0x20000, 16) == 0);       // not mapped
    CHECK(mapped(0x10008, 16) == 0);       // not aligned
    CHECK(mapped(0x10000, ~(size_t)0) == 0);
    auto unknown = [](const void *, Allocation *) { return false; };
    void *out = nullptr;
    CHECK(!map_range(at(0x10000), 16, device_address, unknown, &out));
}

static void check_segments() {
    // 2^32 threads are too many, one block less is not
    CHECK(launch_blocks(64) * 64 < (int64_t)1 << 32 && (launch_blocks(64) + 1) * 64 >= (int64_t)1 << 32);
    CHECK(launch_blocks(256) * 256 < (int64_t)1 << 32 && (launch_blocks(256) + 1) * 256 >= (int64_t)1 << 32);
    auto fit = [](int n, int max_segs, int64_t most, std::initializer_list<int64_t> blocks) {
        return segments_that_fit(n, max_segs, most, [&](int k) { return blocks.begin()[k]; });
    };
    // three segments of 1.9e9 elements: 30M one-wave blocks each, in two launches
    const int64_t b = 30000000;
    CHECK(fit(3, 32, launch_blocks(64), {b, b, b}) == 2);
    CHECK(fit(2, 32, launch_blocks(64), {launch_blocks(64) - 1, 1}) == 2);
    CHECK(fit(2, 32, launch_blocks(64), {launch_blocks(64), 1}) == 1);
    CHECK(fit(2, 32, launch_blocks(256), {launch_blocks(256) - 5, 6}) == 1);
    // a segment that is too large by itself is left to the launch to refuse
    CHECK(fit(2, 32, launch_blocks(64), {launch_blocks(64) + 1, 1}) == 1);
    CHECK(fit(3, 2, launch_blocks(64), {1, 1, 1}) == 2);
    CHECK(fit(1, 32, launch_blocks(64), {1}) == 1);
}

int main() {
    check_segments();
    check_map(0);
    check_map(0x7000000);
    std::printf("ok\n");
    return 0;
}
