// Internal interface between the C ABI (sdp_runtime.hip) and the gfx950
// kernels (sdp_kernels.hip).  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sdp.h"

namespace sdp {

// Result of the norm pass, kept in device memory so that the update kernel
// reads the clip coefficient without a host round trip.
struct NormState {
    double sumsq;
    double norm;
    double clip;
    int32_t nonfinite;
    uint32_t arrived;  // blocks of the finalize that have merged their pairs (the norm pass clears it)
};

// Where the span pairs of a call lie and what to do with their sum: from them
// the finalize makes the norm state, or, for up to kFoldPairs of them, the
// update itself.
struct NormSum {
    const double *pairs;
    int64_t n_pairs;
    double max_grad_norm;
    NormState *ns;      // written
    NormState *mirror;  // NULL, or pinned host memory written too
};

// One launch of the norm pass: `n` elements starting at a tile boundary of
// a segment.  The grid is norm_pairs_per_tile blocks per tile; block b covers
// span b of the segment, kSpan elements (or fewer, or none past the end), and
// writes the pair partials[2b], partials[2b+1], so the tile k of the launch
// owns norm_pairs_per_tile pairs from that many times k.
// When gbar_out is non-null it also stores g_bar there.
struct NormArgs {
    const uint16_t *g[SDP_MAX_RANKS];
    int64_t n;
    double *partials;
    float *gbar_out;
    NormState *ns;  // its arrival count is cleared
    int32_t keep;   // see keep_in_cache
};

// What an update needs beside its segment: the norm state, or the span pairs
// that it sums itself (sum.n_pairs > 0), and the per-step constants, computed
// once on the host in FP64.
struct UpdateConsts {
    const NormState *ns;
    double lr_wd;      // lr * weight_decay
    double beta1, one_minus_beta1;
    double beta2, one_minus_beta2;
    double step_size;  // lr / (1 - beta1^t)
    double inv_bc2;    // 1 / (1 - beta2^t)
    double eps;
    int32_t keep;  // see keep_in_cache
    NormSum sum;
};

// One launch of the fused update over `n` elements.  Gradients come either
// from the R BF16 buffers or, when gbar is non-null, from stored g_bar.
struct UpdateArgs : UpdateConsts {
    float *p, *m, *v;
    uint16_t *pb;
    const uint16_t *g[SDP_MAX_RANKS];
    const float *gbar;
    int64_t n;
    int64_t stride;  // groups between a lane's passes (set by the launch)
};

// One segment of a call on several: its states, its R rank gradients (or
// stored g_bar, which the norm pass writes and the update reads; NULL: none)
// and its size.  The norm pass reads g, gbar and n only.
struct Segment {
    float *p, *m, *v;
    uint16_t *pb;
    const uint16_t *const *g;
    float *gbar;
    int64_t n;
};
// Segments that one launch covers: their pointers travel as kernel arguments,
// which are kept within 4 KiB.
constexpr int kMaxSegsPerLaunch = 32;
constexpr int segs_per_launch(int R) {
    return 3712 / (8 * (R + 8)) < kMaxSegsPerLaunch ? 3712 / (8 * (R + 8)) : kMaxSegsPerLaunch;
}

// One launch of the mean-gradient kernel of the host-update route: g_bar of
// `n` elements from the R BF16 buffers, written to `out` as FP32 or, when
// bf16 is set, rounded to BF16.
struct GbarArgs {
    const uint16_t *g[SDP_MAX_RANKS];
    int64_t n;
    void *out;
    int bf16;
};

// Up to kCopyBatchMax copies of `bytes[k]` bytes from src[k] to dst[k] in
// one launch (the streamed engine's device-to-host copies of a chunk; dst
// may be pinned host memory).  Every dst and src is 16-byte aligned; any
// byte count.
constexpr int kCopyBatchMax = 8;
struct CopyBatch {
    int32_t n;
    char *dst[kCopyBatchMax];
    const char *src[kCopyBatchMax];
    int64_t bytes[kCopyBatchMax];
};

constexpr int kTile = SDP_NORM_TILE;
// Shape of the norm pass for R ranks: spans of kSpan elements, one block of
// kThreads per span, kVec elements per lane and load, kBatch groups of them
// loaded before any is used.  (Rates: TB/s over 419M elements of normal
// gradients, against about 7.1 for plain reads and 6.0 for plain writes.)
//  - Storing g_bar for more than four ranks: the pass is bound by HBM's mix of
//    R read streams and one write stream, which runs faster the closer together
//    the accesses in flight lie: one-wave blocks of one group per lane reach
//    6.58 at R = 8 (6.77 at R = 5, 6.21 at R = 16) where 256-thread blocks over
//    4,096 elements reach 6.05-6.16 (5.83 at R = 16).
//  - Reading alone: large blocks, whose one butterfly is spread over more
//    elements (R = 8: 6.88 against 6.3-6.4 with one-wave blocks; R = 4: 6.79
//    against 6.51).  One rank's 2 bytes per element leave the least time for
//    arithmetic, so its lanes take 32 elements: 6.56, where 16 per lane reach
//    5.5 and 8-byte loads 4.7.
//  - Storing for up to four ranks (streamed mode, bound by the host link) keeps
//    the reading shape's larger spans and so fewer partial pairs.
template <int R, bool STORE>
struct NormShape {
    static constexpr bool kWaveBlocks = STORE && R > 4;
    static constexpr bool kOneWaveOfBlock = false;  // the whole block works on a span
    static constexpr int kThreads = kWaveBlocks ? 64 : 256;
    static constexpr int kVec = R == 1 && !STORE ? 8 : 4;
    static constexpr int kBatch = STORE ? 1 : R == 1 ? 4 : 2;
    static constexpr int kSpan = kWaveBlocks ? 256 : R == 1 && !STORE ? 8192 : 4096;
};
// Partial pairs per norm tile (NormShape<R, store>::kSpan elements each).
constexpr int norm_pairs_per_tile(int R, bool store) {
    return kTile / (store ? (R > 4 ? NormShape<5, true>::kSpan : NormShape<1, true>::kSpan)
                          : (R == 1 ? NormShape<1, false>::kSpan : NormShape<2, false>::kSpan));
}
// Kernels over host memory (streamed mode without copies): as many blocks of
// kHostThreads as have kHostNormBytes or kHostUpdateBytes of loads on their way
// over the link together, in whatever number of ranks and lanes.  Enough of
// them fill the link, and it is bytes that count: some more are 5% slower, and
// many more, at the rate of these again, hold up the chip's other memory
// traffic.  ms over 33.6M elements, R = 4, at 150 / 200 / 240 / 280 / 300 / 320
// / 350 / 450 / 900 KB, the norm pass: 4.73 / 4.69 / 4.69 / 4.67 / 4.67 / 4.71 /
// 4.89 / 4.97 / 4.67 (R = 16 24.3 / 18.9 / 18.8 / 18.7 / 18.8 / 18.8 / 18.7 /
// 19.0 / 18.9); at 130 / 160 / 200 / 222 / 235 / 250 / 350 / 500 / 800 KB, the
// update: 10.3 / 9.34 / 9.24 / 9.16 / 9.16 / 9.62 / 9.84 / 9.29 / 9.24.  (The same
// waves in blocks of 64 or 512 threads: the update 4 to 9% slower.)
// A step of 50.3M elements, R = 4, takes 20.7 ms; beside it, a 4096^3 BF16
// product on another stream (0.14 ms alone) takes 0.23 ms at the median and 0.29
// at most.  With one-wave blocks for the update (128) and a block for every span
// of the norm pass: 21.1 ms, 0.32 and 10.4; through copies: 25.2, 0.15 and 4.3.
constexpr int kHostThreads = 256;
constexpr int kHostNormBytes = 290000;
constexpr int kHostUpdateBytes = 230000;
constexpr int host_blocks(int bytes, int lane_bytes) {
    return bytes / (lane_bytes * kHostThreads) > 1 ? bytes / (lane_bytes * kHostThreads) : 1;
}
// The norm pass there: the spans of NormShape, one wave to a span, with batches
// of about 64 to 128 bytes of loads per lane, so that few waves fill the link.
template <int R, bool STORE>
struct HostNormShape {
    static constexpr bool kOneWaveOfBlock = true;
    static constexpr int kThreads = 64;
    static constexpr int kSpan = NormShape<R, STORE>::kSpan;
    static constexpr int kVec = NormShape<R, STORE>::kVec;
    static constexpr int kBatch = kSpan == 256 ? 1 : kVec == 8 ? 4 : R == 1 ? 8 : R <= 3 ? 4 : R <= 8 ? 2 : 1;
    static constexpr int kBlocks = host_blocks(kHostNormBytes, 2 * R * kVec * kBatch);
};
// The finalize: blocks of kFinalizeThreads merge runs of a multiple of kMergeRun
// pairs each, and the last block to arrive merges their results, so that it is
// one launch at any size: 4.7 us where two launches took 9 (47,104 pairs).  At
// most kMaxMergeBlocks blocks: they count themselves in one after the other,
// about 33 ns apiece (1,675 blocks took 56 us).
constexpr int kFinalizeThreads = 512;
constexpr int kMergeRun = 2048;
constexpr int kMaxMergeBlocks = 128;
// Up to this many pairs every wave of the update sums them itself, behind its
// loads, which saves the finalize's launch: four pairs per lane.  1M elements,
// R = 2 (256 pairs): 18.9 us per step with the finalize, 16.4 without.  Beyond
// it the sum would be repeated by too many waves.
constexpr int kFoldPairs = 256;
constexpr int kUpdateThreads = 64;
// Fused update residency: blocks of one wave, at most kUpdateBlocksPerCU of
// them per compute unit (two or three waves per SIMD).  The update's mix of
// seven read and four write streams runs faster with fewer waves in flight
// than the registers would allow; the cap is imposed with dynamic LDS that
// the kernel does not use (the LDS of a compute unit divided by the cap, per
// block).  Measured, us per step at a cap of 8 / 10 / 11 / 12 / 14:
// Qwen3-8B layer 1275 / 1253 / 1248 / 1249 / 1258, Qwen2.5-72B layer 6955 /
// 6780 / 6723 / 6751 / 6857.  The kernel for several segments looks its
// segment up first and so takes one wave more: 26 segments, R = 1, 3122 / 2952
// / 2863 / 2832 / 2873; nine, R = 4, 361 / 356 / 356 / 359 / 363.
constexpr int kUpdateBlocksPerCU = 11;
constexpr int kUpdateSegmentsBlocksPerCU = 12;
// The norm pass that stores g_bar is capped the same way.  One-wave blocks
// (more than four ranks): the fewer ranks, the more waves it takes to keep the
// same bytes in flight.  Best caps measured: 24 at R = 5, 20 at 6 and 7, 15-16
// at 8 and 9, 13-14 from 10 to 16; no cap costs 2-5%, half the best cap 20-30%.
// 256-thread blocks: 4.  The read-only pass runs uncapped.
constexpr int norm_store_blocks_per_cu(int R) {
    return R > 4 ? (132 / R > 24 ? 24 : 132 / R < 14 ? 14 : 132 / R) : 4;
}
// Its static LDS per block (the block sum of waves 1..3).
constexpr int norm_static_lds(int R, bool store) { return store && R > 4 ? 0 : (256 - 64) * 16; }
constexpr int kUpdVec = 4;  // fused update: elements per lane (8 B of BF16, 16 B of FP32)

// Which accesses of a device-mode call leave the non-temporal hint out, so that
// the 256 MB last-level cache may keep their lines until the update comes for
// them: the norm pass's reads of the gradients or its stores of g_bar, and the
// update's reads of the same.  Plain reads alone are slower (6.5 against 7.1
// TB/s), so this pays only while enough is still there.  us per step, hint /
// norm pass without it / update without it too, by the call's gradient bytes:
//   R = 4:  64 MB 62.9 / 61.3 / 59.4;  128 MB 115.8 / 110.5 / 110.5;  384 MB
//           318 / 307 / 331;  768 MB 630 / 630 / 652;  1.6 GB 1316 / 1335 / 1359
//   R = 2:  64 MB 95.4 / 91.4 / 91.0;  384 MB 516 / 499 / 524;  1.2 GB 1577 / 1580
//   R = 1:  64 MB 159 / 154 / 153;  384 MB 916 / 898 / 920;  1.2 GB 2807 / 2796
//   R = 8:  64 MB 46.1 / 46.1 / 45.3;  200 MB 121.5 / 116.5 / 113.6;  768 MB 432 /
//           426 / 446
//   R = 16: 64 MB 37.3 / 37.7 / 37.1;  200 MB 99.2 / 94.7 / 91.3;  768 MB 346 / 340 /
//           362
// The norm pass's line, 800 MB, is where the gain ends (1 GB, R = 1 to 16: within
// 0.3% of each other).  The update's, 100 MB, lies below where its reads stop
// gaining (between 200 and 384 MB).
// and with stored g_bar (R = 8) by its bytes, hint / stores without / reads too:
//   64 MB 134.7 / 132.7 / 130.5;  96 MB 195.4 / 192.5 / 189.8;  128 MB 254.8 /
//   251.3 / 255.4;  256 MB 497 / 490 / 495;  512 MB 1003 / 1013 / 1048
//   R = 5:  96 MB 175.6 / 172.7 / 168.4;  300 MB 519 / 509 / 536;  512 MB 871 / 870
//   R = 16: 96 MB 262.9 / 262.0 / 258.5;  300 MB 798 / 792 / 821;  400 MB 1050 / 1061
constexpr int kKeepNorm = 1, kKeepUpdate = 2;
constexpr int keep_in_cache(int R, bool store, int64_t elems) {
    return store ? (elems <= 75000000 ? kKeepNorm : 0) | (elems <= 25000000 ? kKeepUpdate : 0)
                 : (elems <= 400000000 / R ? kKeepNorm : 0) | (elems <= 50000000 / R ? kKeepUpdate : 0);
}

hipError_t launch_norm_partials(int R, const NormArgs &a, int store_lds_pad, hipStream_t s);
// The norm pass over n segments (all with gbar or none), in as few launches
// as their arguments allow.  partials: the first pair of the first segment;
// each segment's pairs (norm_pairs_per_tile per tile) follow the previous
// one's.
hipError_t launch_norm_segments(int R, const Segment *segs, int n, double *partials, NormState *ns, int keep,
                                int store_lds_pad, hipStream_t s);
// The same with the gradients in host memory, as the device sees them.
hipError_t launch_norm_segments_host(int R, const Segment *segs, int n, double *partials, NormState *ns,
                                     hipStream_t s);
// The update of n segments (all from gbar or none), likewise.
// lds_pad: for one segment, segments_lds_pad: for several.
hipError_t launch_update_segments(int R, const Segment *segs, int n, const UpdateConsts &c, int lds_pad,
                                  int segments_lds_pad, hipStream_t s);
// merged: room for kMaxMergeBlocks pairs (used when n_pairs > kMergeRun).
hipError_t launch_norm_finalize(const NormSum &sum, double *merged, hipStream_t s);
hipError_t launch_update(int R, UpdateArgs a, int max_blocks, int lds_pad, hipStream_t s);
// The states, and the gradients unless gbar is set, in host memory.
hipError_t launch_update_host(int R, const UpdateArgs &a, hipStream_t s);
// out: pinned host memory as the device sees it.
hipError_t launch_gbar_out(int R, const GbarArgs &a, int max_blocks, hipStream_t s);
hipError_t launch_update_pattern(int R, const UpdateArgs &a, int lds_pad, hipStream_t s);
hipError_t launch_norm_pattern(int R, const NormArgs &a, int store_lds_pad, hipStream_t s);
hipError_t launch_cast_bf16(const float *src, uint16_t *dst, int64_t n, hipStream_t s);
hipError_t launch_copy16(void *dst, const void *src, int64_t n16, int max_blocks, hipStream_t s);
// blocks_per_copy: blocks given to each copy of the batch (at most; fewer
// when a copy is short).
hipError_t launch_copy_batch(const CopyBatch &b, int blocks_per_copy, hipStream_t s);
hipError_t launch_fill_u32(void *dst, int64_t n_words, uint32_t value, hipStream_t s);
// One wave that sleeps `sleeps` times for about 64 x 64 clocks each (a fixed
// count: it always ends); the debug jitter's delay on a stream.
hipError_t launch_sleep(int sleeps, hipStream_t s);

}  // namespace sdp
