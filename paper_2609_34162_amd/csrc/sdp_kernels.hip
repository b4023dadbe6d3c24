// gfx950 kernels of the data-parallel update: norm partials over fixed spans,
// a fixed-order finalize, and the fused aggregate + clip + AdamW + BF16 re-emit pass.  All of them
// are bound by HBM bandwidth and use no MFMA.
// Their lanes move wide accesses: 16-byte (dwordx4) FP32 accesses throughout,
// and BF16 in 16-byte or 8-byte pieces (eight or four elements per lane).
//
// Element arithmetic (the paper names mixed-precision Adam over FP32 master
// weights and moments, fed by the gradient averaged over the ranks, and BF16
// compute weights; the formulas are AdamW with decoupled decay and
// Kingma-Ba bias correction):
//   g_bar = fp32(S / R), S the exact sum of the R BF16 values, rounded once
//   g     = g_bar * c                               (c from the global norm)
//   p1 = p - lr*wd*p ; m' = b1 m + (1-b1) g ; v' = b2 v + (1-b2) g^2
//   p' = p1 - lr/(1-b1^t) * m' / (sqrt(v'/(1-b2^t)) + eps)
// in FP64 registers, each output rounded once to FP32, BF16 from the FP32.
#include "sdp_internal.h"

#include <algorithm>

#include "sdp_limits.h"

namespace sdp {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Streaming accesses: every array of the two passes is touched once per pass,
// so the kernels load and store with the non-temporal hint (the cache does not
// keep the lines), except where keep_in_cache says otherwise.
__device__ __forceinline__ float4 load_nt4(const float *p) {
    const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(p));
    return make_float4(t.x, t.y, t.z, t.w);
}
__device__ __forceinline__ void store_nt4(float *p, float4 v) {
    const f32x4 t = {v.x, v.y, v.z, v.w};
    __builtin_nontemporal_store(t, reinterpret_cast<f32x4 *>(p));
}
__device__ __forceinline__ void store_nt2(uint16_t *p, uint32_t lo, uint32_t hi) {
    const u32x2 t = {lo, hi};
    __builtin_nontemporal_store(t, reinterpret_cast<u32x2 *>(p));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Round to nearest even on the top 16 bits.  NaN: keep sign and top payload
// bits, set the quiet bit (adding the rounding bias could carry a NaN into
// the infinity pattern).  Infinity stays infinity; overflow of the largest
// finite values rounds to infinity as IEEE round-to-nearest does.
__device__ __forceinline__ uint32_t bf16_rne(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x0040u;
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}

__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return bf16_rne(lo) | (bf16_rne(hi) << 16);
}

// fp32(fp64(s / R)) for a finite s.  R a power of two: the product by 1/R is
// exact and equals s / R.  Else Markstein's correction: with y = fp64(1/R) and
// q = fp64(s y), which is within one unit in the last place of s / R, the
// remainder s - R q is exact in one fma and q + y (s - R q), rounded once, is
// the correctly rounded quotient (no underflow here: a nonzero |s| is at
// least 2^-133).  Three operations instead of the divide sequence's eleven.
// An infinite s gives NaN where the quotient is infinite.  That happens to
// lanes whose nonzero values all lie within kExactSpan binades of infinity, and
// nothing shows it: either mean makes the norm NaN, and a call whose norm is not
// finite updates nothing and uses no mean.
template <int R>
__device__ __forceinline__ float mean_of(double s) {
    constexpr double y = 1.0 / (double)R;
    if constexpr ((R & (R - 1)) == 0) {
        return (float)(s * y);
    } else {
        const double q = s * y;
        return (float)__builtin_fma(__builtin_fma(-(double)R, q, s), y, q);
    }
}

// The same for any s, infinities and NaN included.
template <int R>
__device__ __forceinline__ float mean_of_any(double s) {
    return (float)(s / (double)R);
}

// ---------------------------------------------------------------------------
// Mean gradient g_bar = fp32(S / R): S, the exact sum of the R BF16 values,
// divided by R and rounded once.
//
// Fast route.  Summed in FP64 (from +0, in rank order), R BF16 values give S
// exactly when their magnitudes are close enough (span_exact below); then
// fp32(fp64(S / R)) is the single rounding of S / R.  Proof: the two
// roundings differ only if fp64(S / R) is an FP32 midpoint m with S / R != m.
// With 2^E <= S / R < 2^(E+1) that needs |S - R m| <= R 2^(E-53).  S - R m is
// a nonzero multiple of the smaller of S's last-bit weight 2^f and 2^(E-24)
// (the grid of R m); 2^(E-24) exceeds R 2^(E-53) for every R < 2^29, so
// 2^f <= R 2^(E-53), and S / 2^f >= R 2^E / (R 2^(E-53)) = 2^53: S would not
// be an FP64 number.  (Below 2^-126 the FP32 grid is 2^-150 and S's last bit
// weighs at least 2^-133, so the same holds.)
//
// Wide route (magnitudes spread over more binades, which the workloads'
// gradients practically never reach): S is summed exactly as a fixed-point
// integer, rounded to odd at 53 bits (truncated, last bit forced to 1 if
// anything was dropped), and that FP64 value takes the fast route's last two
// steps.  Rounding to odd keeps S on the same side of every number of at most
// 52 significant bits; R times an FP32 value or midpoint has at most 30, so
// fp32 of the quotient is unchanged.

// A lane's values sum exactly in FP64, in any order, when the binade of the
// largest magnitude exceeds that of the smallest nonzero one by at most
// 45 - ceil(log2 R): every value is then a multiple of the smallest one's
// last-bit weight u = 2^(max(e_min, 1) - 134), and every partial sum is
// below R 2^(e_max - 126) <= 2^53 u.
template <int R>
constexpr int kExactSpan = 45 - (R <= 1 ? 0 : R <= 2 ? 1 : R <= 4 ? 2 : R <= 8 ? 3 : 4);

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

// Largest magnitude and smallest nonzero magnitude (minus one) of BF16
// values packed two per word; a zero wraps to 0xffff and so never counts as
// the smallest.
struct Span {
    u16x2 top, low;
};

__device__ __forceinline__ Span span_init() {
    Span s;
    s.top = (u16x2)(0);
    s.low = (u16x2)(0xffff);
    return s;
}

__device__ __forceinline__ void span_add(Span &s, uint32_t word) {
    const u16x2 m = __builtin_bit_cast(u16x2, word & 0x7fff7fffu);
    s.top = __builtin_elementwise_max(s.top, m);
    s.low = __builtin_elementwise_min(s.low, m - (u16x2)(1));
}

template <int R>
__device__ __forceinline__ bool span_exact(const Span &s) {
    const uint32_t top = s.top.x > s.top.y ? s.top.x : s.top.y;
    const uint32_t low = (uint16_t)((s.low.x < s.low.y ? s.low.x : s.low.y) + 1);  // 0: no nonzero value
    const int e_top = (int)(top >> 7);
    const int e_low = (int)(low >> 7) > 1 ? (int)(low >> 7) : 1;
    return e_top - e_low <= kExactSpan<R>;
}

// The wide route's exact sum: S in two's complement in ten 32-bit words,
// bit 0 weighing 2^-133 (the smallest BF16 step).  16 values below 2^128 sum
// below 2^132, so 266 bits with the sign suffice.  The ranks are added one at
// a time, each as a piece of at most 40 bits carried (or borrowed) through
// the words above it: a short loop over few registers.
constexpr int kWideWords = 10;

__device__ __forceinline__ void wide_add(uint32_t (&w)[kWideWords], uint32_t bf16) {
    const uint32_t e = (bf16 >> 7) & 0xffu, f = bf16 & 0x7fu;
    const uint32_t mant = e ? (0x80u | f) : f;  // value = mant * 2^(pos - 133)
    const uint32_t pos = (e ? e : 1u) - 1u;
    const uint64_t piece = (uint64_t)mant << (pos & 31u);
    const uint32_t wi = pos >> 5, plo = (uint32_t)piece, phi = (uint32_t)(piece >> 32);
    const bool sub = (bf16 & 0x8000u) != 0;
    uint32_t carry = 0;  // carry when adding, borrow when subtracting
#pragma unroll
    for (int k = 0; k < kWideWords; ++k) {
        const uint32_t x = k == (int)wi ? plo : k == (int)wi + 1 ? phi : 0u;
        const uint64_t t = sub ? (uint64_t)w[k] - x - carry : (uint64_t)w[k] + x + carry;
        w[k] = (uint32_t)t;
        carry = (uint32_t)(t >> 32) & 1u;
    }
}

// The wide route for one element: rank r's BF16 pattern is g[r][i].
template <int R>
__device__ __forceinline__ float mean_wide(const uint16_t *const *g, int64_t i) {
    uint32_t w[kWideWords];
#pragma unroll
    for (int k = 0; k < kWideWords; ++k) w[k] = 0;
    bool finite = true;
    double s = 0.0;
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
        const uint32_t v = g[r][i];
        finite &= (v & 0x7f80u) != 0x7f80u;
        s += (double)__uint_as_float(v << 16);
        if ((v & 0x7fffu) != 0) wide_add(w, v);
    }
    // NaN or an infinity: the IEEE result of the FP64 sum in rank order
    if (!finite) return mean_of_any<R>(s);
    const bool neg = (w[kWideWords - 1] >> 31) != 0;
    if (neg) {
        uint32_t c = 1;
#pragma unroll
        for (int k = 0; k < kWideWords; ++k) {
            const uint64_t t = (uint64_t)(~w[k]) + c;
            w[k] = (uint32_t)t;
            c = (uint32_t)(t >> 32);
        }
    }
    int top = -1;
#pragma unroll
    for (int k = 0; k < kWideWords; ++k)
        if (w[k]) top = k;
    if (top < 0) return 0.0f;
    // the top three words (zero below word 0) and whether any word under them is nonzero
    uint32_t hw = 0, mw = 0, lw = 0;
    bool below = false;
#pragma unroll
    for (int k = 0; k < kWideWords; ++k) {
        hw = k == top ? w[k] : hw;
        mw = k == top - 1 ? w[k] : mw;
        lw = k == top - 2 ? w[k] : lw;
        below |= (k < top - 2) && w[k] != 0;
    }
    const int sh = __builtin_clz(hw);
    uint64_t hi64 = ((uint64_t)hw << 32) | mw;
    uint32_t rest = lw;
    if (sh) {
        hi64 = (hi64 << sh) | (lw >> (32 - sh));
        rest = lw << sh;
    }
    uint64_t m53 = hi64 >> 11;
    if ((hi64 & 0x7ffu) != 0 || rest != 0 || below) m53 |= 1u;  // round to odd
    const double mag = ldexp((double)m53, 11 + 32 - sh + 32 * (top - 2) - 133);
    return mean_of<R>(neg ? -mag : mag);
}

// The wide route for element i of the R buffers g[r], and for the four
// elements from e0, loading their inputs again (only the rare lanes that
// fail span_exact take it).  Inlined: as a function call it gave every
// kernel a call stack in scratch memory, and the kernels with scratch ran
// three to four times slower (0.67 against 0.23 ms for the Qwen3-8B layer's
// norm pass), since scratch caps the waves in flight.  The ranks are added
// one at a time into ten words, so the route adds few registers.
template <int R>
__device__ __forceinline__ float mean_wide_at(const uint16_t *const *g, int64_t i) {
    return mean_wide<R>(g, i);
}

template <int R>
__device__ __forceinline__ float4 mean_wide_at4(const uint16_t *const *g, int64_t e0) {
    float4 o;
    o.x = mean_wide_at<R>(g, e0);
    o.y = mean_wide_at<R>(g, e0 + 1);
    o.z = mean_wide_at<R>(g, e0 + 2);
    o.w = mean_wide_at<R>(g, e0 + 3);
    return o;
}

// One or two ranks: FP32 gives the singly rounded mean by itself.  A BF16
// value is an FP32 value (adding +0 turns -0 into the definition's +0), and
// half of it is one too, so fma(a, 1/2, b/2) rounds (a + b) / 2 once; b/2
// comes from an fma with +0, so that two zeros of any sign give +0.
__device__ __forceinline__ float mean_fp32(float a) { return a + 0.0f; }
__device__ __forceinline__ float mean_fp32(float a, float b) {
    return __builtin_fmaf(a, 0.5f, __builtin_fmaf(b, 0.5f, 0.0f));
}

// The means of the 2W elements held as BF16 in w[r][0..W-1] (two per word,
// the lower half first), by the fast route; for more than two ranks their
// magnitudes are added to sp, and the means hold only if span_exact<R>(sp)
// (else the caller takes the wide route).
template <int R, int W>
__device__ __forceinline__ void means_of(const uint32_t (&w)[R][W], float *g, Span &sp) {
#pragma unroll
    for (int j = 0; j < W; ++j) {
        if constexpr (R == 1) {
            g[2 * j] = mean_fp32(bf16_lo(w[0][j]));
            g[2 * j + 1] = mean_fp32(bf16_hi(w[0][j]));
        } else if constexpr (R == 2) {
            g[2 * j] = mean_fp32(bf16_lo(w[0][j]), bf16_lo(w[1][j]));
            g[2 * j + 1] = mean_fp32(bf16_hi(w[0][j]), bf16_hi(w[1][j]));
        } else {
            double s_lo = 0.0, s_hi = 0.0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                s_lo += (double)bf16_lo(w[r][j]);
                s_hi += (double)bf16_hi(w[r][j]);
                span_add(sp, w[r][j]);
            }
            g[2 * j] = mean_of<R>(s_lo);
            g[2 * j + 1] = mean_of<R>(s_hi);
        }
    }
}

// Fast route for 2W elements; returns false if the values fail span_exact.
template <int R, int W>
__device__ __forceinline__ bool means_fast(const uint32_t (&w)[R][W], float (&g)[2 * W]) {
    Span sp = span_init();
    means_of<R, W>(w, g, sp);
    if constexpr (R > 2) return span_exact<R>(sp);
    return true;
}

// g_bar of the 4 elements from e0 of the R buffers g[r], whose BF16 words
// (already loaded) are w.
template <int R>
__device__ __forceinline__ void mean4(const uint32_t (&w)[R][2], const uint16_t *const *g, int64_t e0,
                                      float (&out)[4]) {
    const bool fast = means_fast<R, 2>(w, out);
    if constexpr (R > 2) {
        if (__builtin_expect(!fast, 0)) {
            const float4 t = mean_wide_at4<R>(g, e0);
            out[0] = t.x;
            out[1] = t.y;
            out[2] = t.z;
            out[3] = t.w;
        }
    }
}

// g_bar of element i of the R buffers g[r].
template <int R>
__device__ __forceinline__ float mean1(const uint16_t *const *g, int64_t i) {
    uint32_t w[R][1];
#pragma unroll
    for (int r = 0; r < R; ++r) w[r][0] = g[r][i];
    float m[2];
    const bool fast = means_fast<R, 1>(w, m);
    if constexpr (R > 2)
        if (!fast) return mean_wide_at<R>(g, i);
    return m[0];
}

// Double-double accumulation.  S is the sum of the squares of FP32 values,
// each exact in FP64; it is carried as an unevaluated pair hi + lo, hi an FP64
// sum and lo the sum of its rounding errors (relative error below 2^-85, most
// of it from lo's own rounding), so its final rounding to FP64 is that of the
// exact sum, in whatever order and spans it is summed, except when the exact
// sum lies within that distance of an FP64 rounding boundary.  two_sum is
// Knuth's error-free addition.
__device__ __forceinline__ void dd_add(double &hi, double &lo, double x) {
    const double s = hi + x;
    const double bb = s - hi;
    const double e = (hi - (s - bb)) + (x - bb);
    hi = s;
    lo += e;
}

// The lane's partner in step STEP of the butterfly: lane ^ 1, lane ^ 2, then
// (the quads being uniform by then) the mirrored lane of the half row and of
// the row, lane ^ 16 and lane ^ 32.  The first four are register moves within
// a row of 16 lanes (DPP); a shuffle through LDS took about three times as
// long per step.
template <int STEP>
__device__ __forceinline__ int partner_word(int x) {
    if constexpr (STEP == 0) return __builtin_amdgcn_mov_dpp(x, 0xB1, 0xf, 0xf, true);        // quad_perm 1,0,3,2
    else if constexpr (STEP == 1) return __builtin_amdgcn_mov_dpp(x, 0x4E, 0xf, 0xf, true);   // quad_perm 2,3,0,1
    else if constexpr (STEP == 2) return __builtin_amdgcn_mov_dpp(x, 0x141, 0xf, 0xf, true);  // row_half_mirror
    else if constexpr (STEP == 3) return __builtin_amdgcn_mov_dpp(x, 0x140, 0xf, 0xf, true);  // row_mirror
    else return __shfl_xor(x, STEP == 4 ? 16 : 32, 64);
}

template <int STEP>
__device__ __forceinline__ double partner(double x) {
    return __hiloint2double(partner_word<STEP>(__double2hiint(x)), partner_word<STEP>(__double2loint(x)));
}

// Adds a pair to a pair without renormalising: hi stays an FP64 sum, every
// rounding error of which goes to lo.
__device__ __forceinline__ void dd_add_pair(double &hi, double &lo, double bhi, double blo) {
    dd_add(hi, lo, bhi);
    lo += blo;
}

template <int STEP>
__device__ __forceinline__ void wave_merge_step(double &hi, double &lo) {
    const double bh = partner<STEP>(hi), bl = partner<STEP>(lo);
    // the same bits in both partners: every operation here is symmetric
    // (a TwoSum's error term is exact whichever operand comes first)
    const double s = hi + bh;
    const double t = s - hi;
    const double e = (hi - (s - t)) + (bh - t);
    lo = (lo + bl) + e;
    hi = s;
}

__device__ __forceinline__ void wave_merge(double &hi, double &lo) {
    wave_merge_step<0>(hi, lo);
    wave_merge_step<1>(hi, lo);
    wave_merge_step<2>(hi, lo);
    wave_merge_step<3>(hi, lo);
    wave_merge_step<4>(hi, lo);
    wave_merge_step<5>(hi, lo);
}

// Block sum of one pair per thread in a fixed order, valid in thread 0: lane
// l of the first wave adds the pairs of threads l, l + 64, l + 128, ... in
// that order, then a fixed butterfly.  Only one wave runs the butterfly: in
// every wave it cost as much as the sums themselves.
template <int THREADS>
__device__ __forceinline__ void block_merge(double &hi, double &lo) {
    if constexpr (THREADS > 64) {
        __shared__ double2 pairs[THREADS - 64];
        __syncthreads();  // an earlier call's pairs have been read
        if (threadIdx.x >= 64) pairs[threadIdx.x - 64] = make_double2(hi, lo);
        __syncthreads();
        if (threadIdx.x >= 64) return;
#pragma unroll
        for (int k = 0; k < THREADS / 64 - 1; ++k) {
            const double2 b = pairs[k * 64 + threadIdx.x];
            dd_add_pair(hi, lo, b.x, b.y);
        }
    }
    wave_merge(hi, lo);
}

// ---------------------------------------------------------------------------
// Norm partials: a segment is split into spans of NormShape<R, STORE>::kSpan
// elements, block b sums g_bar^2 over span b, and the blocks of a launch
// cover whole tiles (those past the end write a zero pair).  Lane t of a
// block handles the V-element groups b*kSpan/V + k*T + t (k increasing).
// A lane's order, the butterfly and the wave order are fixed, so a span's
// partial depends on its contents only.
//
// Gradients and g_bar move with non-temporal loads and stores, except in calls
// small enough for the last-level cache to keep some of them for the update
// (keep_in_cache).
template <int V, bool NT = true>
__device__ __forceinline__ void load_stream_v(const uint16_t *p, uint32_t (&w)[V / 2]) {
    if constexpr (V == 8) {
        const u32x4 *q = reinterpret_cast<const u32x4 *>(p);
        const u32x4 t = NT ? __builtin_nontemporal_load(q) : *q;
        w[0] = t.x; w[1] = t.y; w[2] = t.z; w[3] = t.w;
    } else {
        const u32x2 *q = reinterpret_cast<const u32x2 *>(p);
        const u32x2 t = NT ? __builtin_nontemporal_load(q) : *q;
        w[0] = t.x; w[1] = t.y;
    }
}

// A power of two that is at least the square of every value of magnitude
// below 2^(e - 126), where e is the biased exponent of the largest magnitude
// among a lane's means.  (The gradients bound their mean too, and their
// largest magnitude is at hand for more than two ranks; but where the ranks
// cancel it lies far above the means, every square falls below the anchor's
// last bit, and the pair degrades to lo alone, one FP64 sum.)
__device__ __forceinline__ double square_anchor(uint32_t e) {
    return __hiloint2double((int)((2u * e + 771u) << 20), 0);  // 2^(2e - 252)
}

// Sum of the squares of one lane's K means, as a pair.  Every square is
// exact in FP64 (48 bits) and at most the anchor, so with the running sum
// started at the anchor each addition is Dekker's Fast2Sum, whose error term
// is exact, and the square itself need not be formed:
// s = fma(g, g, hi), error = fma(g, g, -(s - hi)).  Four operations per value
// where Knuth's TwoSum on the product takes eight.  The anchor leaves hi
// exactly at the end (hi is a multiple of its last bit).  What is rounded is
// lo alone, to 2^-53 of itself: below 2^-90 of the largest square for K <= 32
// (the anchor is at most four times that square, or, among subnormals, has a
// last bit below that of every square).
template <int K>
__device__ __forceinline__ void sum_squares(const float *g, uint32_t e, double &hi, double &lo) {
    const double anchor = square_anchor(e);
    hi = anchor;
    lo = 0.0;
#pragma unroll
    for (int i = 0; i < K; ++i) {
        const double x = (double)g[i];
        const double s = __builtin_fma(x, x, hi);
        lo += __builtin_fma(x, x, hi - s);
        hi = s;
    }
    hi -= anchor;
}

// Biased exponent of the largest magnitude among K FP32 values.
template <int K>
__device__ __forceinline__ uint32_t top_exponent(const float *g) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < K; ++i) m = max(m, __float_as_uint(g[i]) << 1);
    return m >> 24;
}

// The pair of span `blk` of the n-element segment g, and its g_bar if STORE,
// by the T threads of a block, or by one wave of it.  Valid in the first of
// them.
template <int R, bool STORE, bool KEEP, class S>
__device__ __forceinline__ void norm_span(const uint16_t *const *g, int64_t n, int64_t blk, float *gbar, double &hi,
                                          double &lo) {
    constexpr int V = S::kVec, T = S::kThreads, J = S::kBatch;
    const uint32_t lane = S::kOneWaveOfBlock ? threadIdx.x & 63 : threadIdx.x;  // of the span's T
    constexpr int kIters = S::kSpan / (V * T * J);
    static_assert(kIters * V * T * J == S::kSpan, "span must split evenly over the lanes");
    static_assert(kIters <= 32, "one bit per batch of a lane");
    const int64_t span0 = blk * S::kSpan;
    // whole groups of V elements of the segment in this span
    const int64_t left = n - span0;
    const uint32_t groups = left >= S::kSpan ? S::kSpan / V : left > 0 ? (uint32_t)left / V : 0u;
    hi = lo = 0.0;
    uint32_t wide = 0;  // bit `it`: a batch that takes the wide route
    for (int it = 0; it < kIters; ++it) {
        uint32_t raw[J][R][V / 2];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const uint32_t q = (uint32_t)(it * J + j) * T + lane;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (q < groups) {
                    load_stream_v<V, STORE || !KEEP>(g[r] + span0 + q * V, raw[j][r]);
                } else {
#pragma unroll
                    for (int w = 0; w < V / 2; ++w) raw[j][r][w] = 0;
                }
            }
        }
        float m[J * V];
        Span sp = span_init();
#pragma unroll
        for (int j = 0; j < J; ++j) means_of<R, V / 2>(raw[j], m + j * V, sp);
        bool fast = true;
        if constexpr (R > 2) fast = span_exact<R>(sp);
        double bh, bl;
        sum_squares<J * V>(m, top_exponent<J * V>(m), bh, bl);
        if (__builtin_expect(fast, 1)) {
            if constexpr (kIters == 1) {
                hi = bh;
                lo = bl;
            } else {
                dd_add_pair(hi, lo, bh, bl);
            }
            if constexpr (STORE) {
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    const uint32_t q = (uint32_t)(it * J + j) * T + lane;
                    if (q < groups) {
#pragma unroll
                        for (int h = 0; h < V / 4; ++h) {
                            float *at = gbar + span0 + q * V + 4 * h;
                            const float4 x = make_float4(m[j * V + 4 * h], m[j * V + 4 * h + 1], m[j * V + 4 * h + 2],
                                                         m[j * V + 4 * h + 3]);
                            if constexpr (KEEP) *reinterpret_cast<float4 *>(at) = x;
                            else store_nt4(at, x);
                        }
                    }
                }
            }
        } else {
            wide |= 1u << it;
        }
    }
    if constexpr (R > 2) {
        // the batches that failed the span check, in the same order, after the
        // loop, where the wide route's registers do not add to the loop's
        while (__builtin_expect(wide != 0, 0)) {
            const int it = __builtin_ctz(wide);
            wide &= wide - 1;
#pragma unroll 1
            for (int j = 0; j < J * V / 4; ++j) {
                const uint32_t q = (uint32_t)(it * J + j / (V / 4)) * T + lane;
                if (q >= groups) continue;
                const int64_t e0 = span0 + q * V + 4 * (j % (V / 4));
                const float4 t = mean_wide_at4<R>(g, e0);
                dd_add(hi, lo, (double)t.x * (double)t.x);
                dd_add(hi, lo, (double)t.y * (double)t.y);
                dd_add(hi, lo, (double)t.z * (double)t.z);
                dd_add(hi, lo, (double)t.w * (double)t.w);
                if constexpr (STORE) store_nt4(gbar + e0, t);
            }
        }
    }
    // the segment's ragged tail of fewer than V elements, by one lane of its span
    if (lane == 0 && left > 0 && left < S::kSpan) {
        for (int64_t i = span0 + (int64_t)groups * V; i < n; ++i) {
            const float t = mean1<R>(g, i);
            dd_add(hi, lo, (double)t * (double)t);
            if constexpr (STORE) gbar[i] = t;
        }
    }
    block_merge<T>(hi, lo);
}

template <int R, bool WRITE_GBAR, bool KEEP>
__device__ __forceinline__ void norm_partials(const NormArgs &a) {
    double hi, lo;
    norm_span<R, WRITE_GBAR, KEEP, NormShape<R, WRITE_GBAR>>(a.g, a.n, blockIdx.x, a.gbar_out, hi, lo);
    if (threadIdx.x == 0) {
        a.partials[2 * blockIdx.x] = hi;
        a.partials[2 * blockIdx.x + 1] = lo;
        if (blockIdx.x == 0) a.ns->arrived = 0;
    }
}

// Two kernels, here and in the update, because a branch between a plain and a
// non-temporal access is merged into one plain access by the compiler.
template <int R, bool WRITE_GBAR>
__global__ __launch_bounds__((NormShape<R, WRITE_GBAR>::kThreads)) void k_norm_partials(NormArgs a) {
    norm_partials<R, WRITE_GBAR, false>(a);
}

template <int R, bool WRITE_GBAR>
__global__ __launch_bounds__((NormShape<R, WRITE_GBAR>::kThreads)) void k_norm_partials_keep(NormArgs a) {
    norm_partials<R, WRITE_GBAR, true>(a);
}

// ---------------------------------------------------------------------------
// Several segments in one launch.  A call's segments are often small (the
// tensors of a layer, the layers of a small model): a launch each left the
// chip idle in every ragged last wave of blocks and 2-8 us between kernels,
// and cost the host 2.3 us each.  Measured with one launch per segment and
// with this one: nine tensors, 48M elements, R = 4, 400 and 356 us; 26
// segments, 613M elements, R = 1, 3115 and 2832 us; four tensors of 231,084
// elements in all, 70 and 37 us.
template <int R>
struct SegEntry {  // one run of scalar loads
    int64_t end;    // first block after the segment
    int64_t first;  // its first block
    float *p, *m, *v;
    uint16_t *pb;
    float *gbar;
    int64_t n;
    const uint16_t *g[R];
};

// The segment of a block is looked up in a map of up to 256 runs of 2^shift
// blocks, four one-byte entries per word: the segment of the run's first
// block, from which the few blocks of later segments step on.  Two scalar
// loads deep, against one for a single segment; comparing the block with
// every segment's first one instead held each wave back by 0.3 us, 10% of
// its life, and the update with it.
constexpr int kSegMapRuns = 256;
template <int R>
struct SegTable {
    static constexpr int kSegs = segs_per_launch(R);
    uint32_t map[kSegMapRuns / 4];
    uint32_t shift;
    SegEntry<R> seg[kSegs];
};

// With the largest arguments beside it (the update's), within the 4 KiB that
// segs_per_launch plans for.
template <int R>
constexpr bool kTableFits = sizeof(SegTable<R>) + sizeof(UpdateConsts) <= 4096;

template <int R>
__device__ __forceinline__ const SegEntry<R> &segment_of(const SegTable<R> &t, uint32_t b) {
    const uint32_t run = b >> t.shift;
    uint32_t s = t.map[run / 4] >> (run % 4 * 8) & 0xffu;
    while (__builtin_expect(b >= t.seg[s].end, 0)) ++s;
    return t.seg[s];
}

template <int R, bool WRITE_GBAR, bool KEEP>
__global__ __launch_bounds__((NormShape<R, WRITE_GBAR>::kThreads)) void k_norm_segments(SegTable<R> t,
                                                                                      double *partials,
                                                                                      NormState *ns) {
    const SegEntry<R> &e = segment_of<R>(t, blockIdx.x);
    double hi, lo;
    norm_span<R, WRITE_GBAR, KEEP, NormShape<R, WRITE_GBAR>>(e.g, e.n, blockIdx.x - e.first, e.gbar, hi, lo);
    if (threadIdx.x == 0) {
        partials[2 * (int64_t)blockIdx.x] = hi;
        partials[2 * (int64_t)blockIdx.x + 1] = lo;
        if (blockIdx.x == 0) ns->arrived = 0;
    }
}

// The same over host memory (streamed mode without copies): the waves of a few
// blocks walk the spans, one wave to a span.  Bound by the link.  Blocks for
// every span under the stored pass's residency pad, which filled the LDS of
// every compute unit, were no faster and kept the kernels of other streams
// waiting: a 4096^3 BF16 product of 0.14 ms took up to the whole pass, 14.3 ms
// at 50M elements and R = 8.
template <int R, bool WRITE_GBAR>
__global__ __launch_bounds__(kHostThreads) void k_norm_segments_host(SegTable<R> t, uint32_t spans, double *partials,
                                                                      NormState *ns) {
    const uint32_t waves = gridDim.x * (kHostThreads / 64);
    uint32_t at = blockIdx.x * (kHostThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    // each round of `waves` spans goes round the waves one further on: where the
    // segments are small, their one span with elements lies at every 16th place
    for (uint32_t first = 0; first < spans; first += waves, at = at + 1 == waves ? 0 : at + 1) {
        const uint32_t b = first + at;
        if (b >= spans) continue;
        const SegEntry<R> &e = segment_of<R>(t, b);
        using S = HostNormShape<R, WRITE_GBAR>;
        double hi = 0.0, lo = 0.0;
        if ((b - e.first) * S::kSpan < e.n)  // most spans of a small segment's tile lie past its end
            norm_span<R, WRITE_GBAR, false, S>(e.g, e.n, b - e.first, e.gbar, hi, lo);
        if ((threadIdx.x & 63) == 0) {
            partials[2 * (int64_t)b] = hi;
            partials[2 * (int64_t)b + 1] = lo;
            if (b == 0) ns->arrived = 0;
        }
    }
}

// ---------------------------------------------------------------------------
// The norm from the span pairs.

// The norm state of the sum of squares hi + lo, written where it is wanted.
__device__ __forceinline__ NormState norm_state(double hi, double lo, double max_grad_norm) {
    NormState st;
    st.sumsq = hi + lo;
    st.norm = sqrt(st.sumsq);
    st.nonfinite = !isfinite(st.sumsq);
    st.clip = 1.0;
    if (max_grad_norm > 0.0 && !st.nonfinite) {
        st.clip = max_grad_norm / (st.norm + 1e-6);
        if (st.clip > 1.0) st.clip = 1.0;
    }
    st.arrived = 0;
    return st;
}

// Sum of up to kFoldPairs pairs by one wave, the same bits in every lane: lane
// l adds pairs l, l + 64, l + 128, l + 192, then the butterfly.
__device__ __forceinline__ void fold_pairs(const double *pairs, int64_t n_pairs, double &hi, double &lo) {
    const double2 *p = reinterpret_cast<const double2 *>(pairs);
    const int lane = threadIdx.x & 63;
    double2 b[kFoldPairs / 64];
#pragma unroll
    for (int k = 0; k < kFoldPairs / 64; ++k)
        b[k] = k * 64 + lane < n_pairs ? p[k * 64 + lane] : make_double2(0.0, 0.0);
    hi = b[0].x;
    lo = b[0].y;
#pragma unroll
    for (int k = 1; k < kFoldPairs / 64; ++k) dd_add_pair(hi, lo, b[k].x, b[k].y);
    wave_merge(hi, lo);
}

// Up to kFoldPairs pairs: one wave, as the update does.  Up to kMergeRun: one
// block.  More: block b merges the `run` pairs from b * run (a multiple of
// kMergeRun), thread t of it t + kFinalizeThreads * j in increasing j, into
// merged pair b, and the last block to arrive merges those in the same way; no
// block waits for another.
// The merged pairs and the count pass between blocks on different XCDs, so
// they move by device-scope atomics.  Bound by the latency of its loads and of
// the few dependent steps, not by any rate.
__global__ __launch_bounds__(kFinalizeThreads) void k_norm_finalize(NormSum sum, int64_t run,
                                                                      double *__restrict__ merged) {
    constexpr int T = kFinalizeThreads;
    double hi = 0.0, lo = 0.0;
    if (sum.n_pairs <= kFoldPairs) {
        if (threadIdx.x >= 64) return;
        fold_pairs(sum.pairs, sum.n_pairs, hi, lo);
    } else {
        const double2 *p = reinterpret_cast<const double2 *>(sum.pairs);
        for (int64_t at = 0; at < run; at += kMergeRun) {
            const int64_t base = (int64_t)blockIdx.x * run + at + threadIdx.x;
            double2 b[kMergeRun / T];
#pragma unroll
            for (int j = 0; j < kMergeRun / T; ++j)
                b[j] = base + j * T < sum.n_pairs ? p[base + j * T] : make_double2(0.0, 0.0);
#pragma unroll
            for (int j = 0; j < kMergeRun / T; ++j) dd_add_pair(hi, lo, b[j].x, b[j].y);
        }
        block_merge<T>(hi, lo);
        if (gridDim.x > 1) {
            __shared__ bool last;
            if (threadIdx.x == 0) {
                __hip_atomic_store(merged + 2 * blockIdx.x, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(merged + 2 * blockIdx.x + 1, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = __hip_atomic_fetch_add(&sum.ns->arrived, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
                       gridDim.x - 1;
            }
            __syncthreads();
            if (!last) return;
            hi = lo = 0.0;
            for (uint32_t i = threadIdx.x; i < gridDim.x; i += T)
                dd_add_pair(hi, lo, __hip_atomic_load(merged + 2 * i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                            __hip_atomic_load(merged + 2 * i + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            block_merge<T>(hi, lo);
        }
    }
    if (threadIdx.x == 0) {
        const NormState st = norm_state(hi, lo, sum.max_grad_norm);
        *sum.ns = st;
        if (sum.mirror) *sum.mirror = st;
    }
}

// ---------------------------------------------------------------------------
// Fused update.

struct Consts {
    double c, lr_wd, beta1, omb1, beta2, omb2, step_size, inv_bc2, eps;
    int nonfinite;
};

// p1, m' and v' are each rounded after every product and sum, in the order
// of their definition (no fused multiply-add).  m' cancels where b1*m is
// close to -(1-b1)*g -- common, since the inputs sit on the coarse BF16 grid
// -- and there a single-rounding fma and a two-rounding evaluation differ by
// a large relative amount of a result that is pure rounding noise.  Fixing
// the order makes m' (and v', p1) the same bits as the definition's.
__device__ __forceinline__ void moments(double pd, double md, double vd, double g, const Consts &k,
                                        double &p1, double &m1, double &v1) {
#pragma clang fp contract(off)
    p1 = pd - k.lr_wd * pd;
    m1 = k.beta1 * md + k.omb1 * g;
    v1 = k.beta2 * vd + k.omb2 * (g * g);
}

__device__ __forceinline__ void adamw(float &p, float &m, float &v, float g_bar, const Consts &k) {
#pragma clang fp contract(off)
    const double g = (double)g_bar * k.c;
    double p1, m1, v1;
    moments((double)p, (double)m, (double)v, g, k, p1, m1, v1);
    const double denom = sqrt(v1 * k.inv_bc2) + k.eps;
    const double pn = p1 - k.step_size * (m1 / denom);
    p = (float)pn;
    m = (float)m1;
    v = (float)v1;
}

// The norm state comes through scalar loads (an earlier kernel wrote it and
// no block of this one does), or (FOLD) the wave sums the span pairs itself,
// and the grid's first wave writes the norm state.  All lanes of the wave call
// it together.
template <bool FOLD>
__device__ __forceinline__ Consts load_consts(const UpdateConsts &a) {
    Consts k;
    if constexpr (FOLD) {
        double hi, lo;
        fold_pairs(a.sum.pairs, a.sum.n_pairs, hi, lo);
        const NormState st = norm_state(hi, lo, a.sum.max_grad_norm);
        k.c = st.clip;
        k.nonfinite = __builtin_amdgcn_readfirstlane(st.nonfinite);
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            *a.sum.ns = st;
            if (a.sum.mirror) *a.sum.mirror = st;
        }
    } else {
        uintptr_t at = (uintptr_t)a.ns;
        // behind the loads before it: waiting for the norm state first would
        // add a memory latency to every wave
        asm volatile("" : "+s"(at)::"memory");
        const auto *ns = (const __attribute__((address_space(4))) NormState *)at;
        k.nonfinite = ns->nonfinite;
        k.c = ns->clip;
    }
    k.lr_wd = a.lr_wd;
    k.beta1 = a.beta1;
    k.omb1 = a.one_minus_beta1;
    k.beta2 = a.beta2;
    k.omb2 = a.one_minus_beta2;
    k.step_size = a.step_size;
    k.inv_bc2 = a.inv_bc2;
    k.eps = a.eps;
    return k;
}

// One wave's part of a segment: lane l takes the 4-element groups w0 + l,
// w0 + stride + l, ..., and lane 0 of the segment's first wave its ragged tail
// of fewer than 4 elements.  Each access of the wave is one contiguous run
// (1 KB of every FP32 array, 512 B of every BF16 one).
// Every access to the states is non-temporal: under the residency cap this
// measured about 5% faster than plain accesses.
template <int R, bool CACHED, bool FOLD, bool KEEP>
__device__ __forceinline__ void update_groups(float *__restrict__ P, float *__restrict__ M, float *__restrict__ V,
                                              uint16_t *__restrict__ PB, const uint16_t *const *grads,
                                              const float *__restrict__ GB, int64_t n, int64_t w0, int64_t stride,
                                              const UpdateConsts &a) {
    const int64_t groups = n / kUpdVec;
    const int lane = threadIdx.x & 63;
    Consts k;
    for (int64_t w = w0;;) {
        const bool has = w + lane < groups;
        const int64_t e0 = (w + lane) * kUpdVec;
        float4 gb, pv, mv, vv;
        uint32_t raw[R][2];
        if (has) {
            if constexpr (CACHED) {
                gb = KEEP ? *reinterpret_cast<const float4 *>(GB + e0) : load_nt4(GB + e0);
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) load_stream_v<4, !KEEP>(grads[r] + e0, raw[r]);
            }
            pv = load_nt4(P + e0);
            mv = load_nt4(M + e0);
            vv = load_nt4(V + e0);
        }
        k = load_consts<FOLD>(a);
        if (has) {
            float g[kUpdVec];
            if constexpr (CACHED) {
                g[0] = gb.x; g[1] = gb.y; g[2] = gb.z; g[3] = gb.w;
            } else {
                mean4<R>(raw, grads, e0, g);
            }
            float *pf = &pv.x, *mf = &mv.x, *vf = &vv.x;
#pragma unroll
            for (int e = 0; e < kUpdVec; ++e) adamw(pf[e], mf[e], vf[e], g[e], k);
            // a non-finite norm is acted on here and not before the loads,
            // which would then wait for the norm state: the results pass
            // through an empty statement, so that the compiler cannot move
            // the branch up
            int skip = k.nonfinite;
            asm volatile("" : "+s"(skip) : "v"(pv.x), "v"(pv.y), "v"(pv.z), "v"(pv.w), "v"(mv.x), "v"(mv.y),
                         "v"(mv.z), "v"(mv.w), "v"(vv.x), "v"(vv.y), "v"(vv.z), "v"(vv.w));
            if (!skip) {
                store_nt4(P + e0, pv);
                store_nt4(M + e0, mv);
                store_nt4(V + e0, vv);
                store_nt2(PB + e0, pack_bf16(pf[0], pf[1]), pack_bf16(pf[2], pf[3]));
            }
        }
        if (stride >= groups - w) break;
        w += stride;
    }
    if (w0 == 0 && lane == 0 && !k.nonfinite) {
        for (int64_t i = groups * kUpdVec; i < n; ++i) {
            float gb;
            if constexpr (CACHED) gb = GB[i];
            else gb = mean1<R>(grads, i);
            float p = P[i], m = M[i], v = V[i];
            adamw(p, m, v, gb, k);
            P[i] = p; M[i] = m; V[i] = v;
            PB[i] = (uint16_t)bf16_rne(p);
        }
    }
}

template <int R, bool CACHED>
__global__ __launch_bounds__(kUpdateThreads) void k_update(UpdateArgs a) {
    update_groups<R, CACHED, false, false>(a.p, a.m, a.v, a.pb, a.g, a.gbar, a.n,
                                           (int64_t)blockIdx.x * kUpdateThreads, a.stride, a);
}

template <int R, bool CACHED>
__global__ __launch_bounds__(kUpdateThreads) void k_update_keep(UpdateArgs a) {
    update_groups<R, CACHED, false, true>(a.p, a.m, a.v, a.pb, a.g, a.gbar, a.n,
                                          (int64_t)blockIdx.x * kUpdateThreads, a.stride, a);
}

// The update of a segment in host memory, by the waves of a few blocks.  Bound
// by the link.
template <int R, bool CACHED>
__global__ __launch_bounds__(kHostThreads) void k_update_host(UpdateArgs a) {
    const int64_t wave = (int64_t)blockIdx.x * (kHostThreads / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    update_groups<R, CACHED, false, false>(a.p, a.m, a.v, a.pb, a.g, a.gbar, a.n, wave * 64, a.stride, a);
}

// The update of several segments: block b handles the 64 groups from
// 64 * (b - first) of its segment.
template <int R, bool CACHED, bool FOLD, bool KEEP>
__global__ __launch_bounds__(kUpdateThreads) void k_update_segments(SegTable<R> t, UpdateConsts c) {
    const SegEntry<R> &e = segment_of<R>(t, blockIdx.x);
    update_groups<R, CACHED, FOLD, KEEP>(e.p, e.m, e.v, e.pb, e.g, e.gbar, e.n, (blockIdx.x - e.first) * kUpdateThreads,
                             (int64_t)1 << 62, c);
}

// ---------------------------------------------------------------------------
// Measurement: the fused update's memory access pattern with trivial
// arithmetic (integer and FP32 adds instead of the FP64 AdamW), the same
// loads, stores, widths and lane mapping, from the R gradients or (CACHED)
// from stored g_bar.  Its rate is the ceiling that the update's own traffic
// mix allows on this part.  Overwrites the states.

template <int R, bool CACHED>
__global__ __launch_bounds__(kUpdateThreads) void k_update_pattern(UpdateArgs a) {
    float *__restrict__ P = a.p;
    float *__restrict__ M = a.m;
    float *__restrict__ V = a.v;
    uint16_t *__restrict__ PB = a.pb;
    const int64_t n = a.n;
    const int64_t groups = n / kUpdVec;
    const int64_t gid = (int64_t)blockIdx.x * kUpdateThreads + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kUpdateThreads;
    for (int64_t q = gid; q < groups; q += stride) {
        const int64_t e0 = q * kUpdVec;
        uint32_t x = 0;
        if constexpr (CACHED) {
            const float4 t = load_nt4(a.gbar + e0);
            x = __float_as_uint(t.x) ^ __float_as_uint(t.y) ^ __float_as_uint(t.z) ^ __float_as_uint(t.w);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint32_t w[2];
                load_stream_v<4>(a.g[r] + e0, w);
                x ^= w[0] ^ w[1];
            }
        }
        const float gx = __uint_as_float((x & 0x007fffffu) | 0x3f800000u);
        float4 pv = load_nt4(P + e0), mv = load_nt4(M + e0), vv = load_nt4(V + e0);
        float *pf = &pv.x, *mf = &mv.x, *vf = &vv.x;
#pragma unroll
        for (int e = 0; e < kUpdVec; ++e) {
            pf[e] += gx;
            mf[e] += pf[e];
            vf[e] += mf[e];
        }
        store_nt4(P + e0, pv);
        store_nt4(M + e0, mv);
        store_nt4(V + e0, vv);
        store_nt2(PB + e0, (__float_as_uint(pf[0]) >> 16) | (__float_as_uint(pf[1]) & 0xffff0000u),
                  (__float_as_uint(pf[2]) >> 16) | (__float_as_uint(pf[3]) & 0xffff0000u));
    }
}

// ---------------------------------------------------------------------------
// Measurement: the g_bar-storing norm pass's memory access pattern with
// trivial arithmetic (xor of the ranks' bits instead of the exact mean and
// the double-double sum of squares): the same grid, lane mapping, loads,
// 16-byte stores and span pairs, under the same residency cap.  Its rate is
// the ceiling that the pass's own traffic mix allows on this part.  The
// ragged tail of fewer than 4 elements is left out.

template <int R>
__global__ __launch_bounds__((NormShape<R, true>::kThreads)) void k_norm_pattern(NormArgs a) {
    using S = NormShape<R, true>;
    constexpr int V = S::kVec, T = S::kThreads;
    static_assert(V == 4, "one 16-byte store per group");
    const int64_t span0 = (int64_t)blockIdx.x * S::kSpan;
    const int64_t left = a.n - span0;
    const uint32_t groups = left >= S::kSpan ? S::kSpan / V : left > 0 ? (uint32_t)left / V : 0u;
    uint32_t acc = 0;
    for (uint32_t q = threadIdx.x; q < groups; q += T) {
        uint32_t x0 = 0, x1 = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t w[2];
            load_stream_v<V>(a.g[r] + span0 + q * V, w);
            x0 ^= w[0];
            x1 ^= w[1];
        }
        store_nt4(a.gbar_out + span0 + q * V, make_float4(bf16_lo(x0), bf16_hi(x0), bf16_lo(x1), bf16_hi(x1)));
        acc ^= x0 ^ x1;
    }
    double hi = (double)acc, lo = 0.0;
    block_merge<T>(hi, lo);
    if (threadIdx.x == 0) {
        a.partials[2 * blockIdx.x] = hi;
        a.partials[2 * blockIdx.x + 1] = lo;
    }
}

// ---------------------------------------------------------------------------
// Mean gradient for the host-update route: g_bar of a piece, FP32 or rounded
// to BF16, written straight into a pinned host buffer, so bound by the link's
// device-to-host direction.  A wave's stores are one contiguous run of 1 KB
// (four FP32 or eight BF16 results per lane): the link moves whole runs, and
// interleaved half-lines would cost it twice the requests.  The rank gradients
// are read once and not reused (non-temporal).  Route step of the Qwen3-8B
// layer, through a device slot and a copy / written directly: 18.55 / 18.25 ms
// with the FP32 mean gradient, 16.9 / 16.3 ms with the BF16 one.

template <int R, bool BF16>
__global__ __launch_bounds__(256) void k_gbar_out(GbarArgs a) {
    constexpr int V = BF16 ? 8 : 4;
    const int64_t n = a.n;
    const int64_t groups = n / V;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t q = gid; q < groups; q += stride) {
        uint32_t raw[R][V / 2];
#pragma unroll
        for (int r = 0; r < R; ++r) load_stream_v<V>(a.g[r] + q * V, raw[r]);
        float g[V];
#pragma unroll
        for (int h = 0; h < V / 4; ++h) {
            uint32_t w[R][2];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                w[r][0] = raw[r][2 * h];
                w[r][1] = raw[r][2 * h + 1];
            }
            float g4[4];
            mean4<R>(w, a.g, q * V + 4 * h, g4);
#pragma unroll
            for (int e = 0; e < 4; ++e) g[4 * h + e] = g4[e];
        }
        if constexpr (BF16) {
            const u32x4 b = {pack_bf16(g[0], g[1]), pack_bf16(g[2], g[3]), pack_bf16(g[4], g[5]), pack_bf16(g[6], g[7])};
            __builtin_nontemporal_store(b, reinterpret_cast<u32x4 *>(a.out) + q);
        } else {
            store_nt4(reinterpret_cast<float *>(a.out) + q * 4, make_float4(g[0], g[1], g[2], g[3]));
        }
    }
    if (gid == 0) {
        for (int64_t i = groups * V; i < n; ++i) {
            const float g = mean1<R>(a.g, i);
            if constexpr (BF16) reinterpret_cast<uint16_t *>(a.out)[i] = (uint16_t)bf16_rne(g);
            else reinterpret_cast<float *>(a.out)[i] = g;
        }
    }
}

// ---------------------------------------------------------------------------
// Small helpers.

// Four elements per lane, non-temporal, so that a wave's load is one run of
// 1 KB: 419M elements in 402 us, 6.25 TB/s (eight per lane in two 16-byte loads
// 32 bytes apart: 449 us).
__global__ __launch_bounds__(256) void k_cast_bf16(const float *__restrict__ src,
                                                   uint16_t *__restrict__ dst, int64_t n) {
    const int64_t groups = n / 4;
    const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t q = gid; q < groups; q += stride) {
        const float4 x = load_nt4(src + q * 4);
        store_nt2(dst + q * 4, pack_bf16(x.x, x.y), pack_bf16(x.z, x.w));
    }
    if (gid == 0)
        for (int64_t i = groups * 4; i < n; ++i) dst[i] = (uint16_t)bf16_rne(src[i]);
}

__global__ __launch_bounds__(256) void k_copy16(uint4 *__restrict__ dst, const uint4 *__restrict__ src,
                                                int64_t n16) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t *__restrict__ dst, int64_t n_words, uint32_t value) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t n4 = n_words / 4;
    uint4 v4 = make_uint4(value, value, value, value);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n4; i += stride)
        reinterpret_cast<uint4 *>(dst)[i] = v4;
    if (blockIdx.x == 0 && threadIdx.x == 0)
        for (int64_t i = n4 * 4; i < n_words; ++i) dst[i] = value;
}

// ceil(a / b) for a >= 0, b > 0, without overflow near the int64 limit
inline int64_t cdiv(int64_t a, int64_t b) { return a / b + (a % b != 0); }

template <int R, bool STORE>
hipError_t norm_rs(const NormArgs &a, int lds_pad, hipStream_t s) {
    using S = NormShape<R, STORE>;
    static_assert(kTile / S::kSpan == norm_pairs_per_tile(R, STORE), "the host's pair count");
    const dim3 grid((uint32_t)(cdiv(a.n, kTile) * (kTile / S::kSpan))), block(S::kThreads);
    if (a.keep)
        hipLaunchKernelGGL((k_norm_partials_keep<R, STORE>), grid, block, lds_pad, s, a);
    else
        hipLaunchKernelGGL((k_norm_partials<R, STORE>), grid, block, lds_pad, s, a);
    return hipGetLastError();
}

template <int R>
hipError_t norm_r(const NormArgs &a, int store_lds_pad, hipStream_t s) {
    return a.gbar_out ? norm_rs<R, true>(a, store_lds_pad, s) : norm_rs<R, false>(a, 0, s);
}

template <int R, bool CACHED>
hipError_t update_rc(const UpdateArgs &a, int64_t blocks, int lds_pad, hipStream_t s) {
    const dim3 grid((uint32_t)blocks), block(kUpdateThreads);
    if (a.keep)
        hipLaunchKernelGGL((k_update_keep<R, CACHED>), grid, block, lds_pad, s, a);
    else
        hipLaunchKernelGGL((k_update<R, CACHED>), grid, block, lds_pad, s, a);
    return hipGetLastError();
}

template <int R>
hipError_t update_r(const UpdateArgs &a, int64_t blocks, int lds_pad, hipStream_t s) {
    return a.gbar ? update_rc<1, true>(a, blocks, lds_pad, s) : update_rc<R, false>(a, blocks, lds_pad, s);
}

// Block counts of one segment in the batched launches.
int64_t update_blocks(int64_t n) {
    const int64_t b = cdiv(n / kUpdVec, kUpdateThreads);
    return b < 1 ? 1 : b;
}

// Fills `t` from segs[0 .. n): as many segments as fit the table and have at
// most max_blocks blocks; returns how many, and the blocks they need.
template <int R, class F>
int fill_table(SegTable<R> &t, const Segment *segs, int n, bool cached_only, int64_t max_blocks, F blocks_of,
               int64_t *blocks) {
    const int fit = sdprt::segments_that_fit(n, SegTable<R>::kSegs, max_blocks,
                                             [&](int k) { return blocks_of(segs[k].n); });
    static_assert(kTableFits<R>, "the kernel arguments of a launch over several segments");
    *blocks = 0;
    for (int k = 0; k < fit; ++k) {
        const int64_t b = blocks_of(segs[k].n);
        SegEntry<R> &e = t.seg[k];
        e.p = segs[k].p;
        e.m = segs[k].m;
        e.v = segs[k].v;
        e.pb = segs[k].pb;
        e.gbar = segs[k].gbar;
        e.n = segs[k].n;
        e.first = *blocks;
        for (int r = 0; r < R && !cached_only; ++r) e.g[r] = segs[k].g[r];
        *blocks += b;
        e.end = *blocks;
    }
    while ((*blocks - 1) >> t.shift >= kSegMapRuns) ++t.shift;
    for (int run = 0, at = 0; run < kSegMapRuns && (int64_t)run << t.shift < *blocks; ++run) {
        while (t.seg[at].end <= (int64_t)run << t.shift) ++at;
        t.map[run / 4] |= (uint32_t)at << (run % 4 * 8);
    }
    return fit;
}

template <int R>
hipError_t norm_segments_r(const Segment *segs, int n, double *partials, NormState *ns, int keep, int store_lds_pad,
                           hipStream_t s) {
    const bool store = segs[0].gbar != nullptr;
    const int ppt = norm_pairs_per_tile(R, store);
    for (int k = 0; k < n;) {
        if (n - k == 1) {
            NormArgs a{};
            for (int r = 0; r < R; ++r) a.g[r] = segs[k].g[r];
            a.n = segs[k].n;
            a.partials = partials;
            a.gbar_out = segs[k].gbar;
            a.ns = ns;
            a.keep = keep;
            return norm_r<R>(a, store_lds_pad, s);
        }
        SegTable<R> t{};
        int64_t blocks = 0;
        const int threads = store ? NormShape<R, true>::kThreads : NormShape<R, false>::kThreads;
        const int done = fill_table<R>(t, segs + k, n - k, false, sdprt::launch_blocks(threads),
                                       [&](int64_t e) { return cdiv(e, kTile) * ppt; }, &blocks);
        const dim3 grid((uint32_t)blocks), block(threads);
        const int lds_pad = store ? store_lds_pad : 0;
        auto kernel = store ? (keep ? k_norm_segments<R, true, true> : k_norm_segments<R, true, false>)
                            : (keep ? k_norm_segments<R, false, true> : k_norm_segments<R, false, false>);
        hipLaunchKernelGGL(kernel, grid, block, lds_pad, s, t, partials, ns);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        partials += 2 * blocks;
        k += done;
    }
    return hipSuccess;
}

template <int R>
hipError_t norm_segments_host_r(const Segment *segs, int n, double *partials, NormState *ns, hipStream_t s) {
    static_assert(HostNormShape<R, true>::kSpan == NormShape<R, true>::kSpan &&
                      HostNormShape<R, false>::kSpan == NormShape<R, false>::kSpan,
                  "the pairs of every pass lie alike");
    const bool store = segs[0].gbar != nullptr;
    const int ppt = norm_pairs_per_tile(R, store);
    auto kernel = store ? k_norm_segments_host<R, true> : k_norm_segments_host<R, false>;
    const int most = store ? HostNormShape<R, true>::kBlocks : HostNormShape<R, false>::kBlocks;
    for (int k = 0; k < n;) {
        SegTable<R> t{};
        int64_t spans = 0;
        // the kernel counts spans in 32 bits
        k += fill_table<R>(t, segs + k, n - k, false, INT32_MAX, [&](int64_t e) { return cdiv(e, kTile) * ppt; }, &spans);
        if (spans > INT32_MAX) return hipErrorInvalidConfiguration;
        const int64_t blocks = std::min<int64_t>(cdiv(spans, kHostThreads / 64), most);
        hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(kHostThreads), 0, s, t, (uint32_t)spans, partials, ns);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        partials += 2 * spans;
    }
    return hipSuccess;
}

template <int R>
hipError_t update_host_r(UpdateArgs a, hipStream_t s) {
    // a lane's loads from the host: the three states, and the gradients unless
    // g_bar is stored.  (Sixteen ranks' gradients take twice the blocks: 33.6M
    // elements, ms at 230 / 300 / 500 / 1,500 KB: R = 16 31.6 / 28.4 / 25.8 / 25.7,
    // R = 15 24.9 / 24.5 / 25.4 / 24.5, R = 8 16.5 / 16.6 / 17.6 / 16.5.)
    const int most = host_blocks(a.gbar || R < 16 ? kHostUpdateBytes : 500000, 3 * 16 + (a.gbar ? 0 : 8 * R));
    const int64_t blocks = std::min<int64_t>(std::max<int64_t>(cdiv(a.n / kUpdVec, kHostThreads), 1), most);
    a.stride = blocks * kHostThreads;
    if (a.gbar)
        hipLaunchKernelGGL((k_update_host<1, true>), dim3((uint32_t)blocks), dim3(kHostThreads), 0, s, a);
    else
        hipLaunchKernelGGL((k_update_host<R, false>), dim3((uint32_t)blocks), dim3(kHostThreads), 0, s, a);
    return hipGetLastError();
}

// R ranks, or (CACHED) the stored g_bar, where R = 1 stands for any number.
template <int R, bool CACHED>
hipError_t update_segments_r(const Segment *segs, int n, const UpdateConsts &c, int lds_pad, int segments_lds_pad,
                             hipStream_t s) {
    for (int k = 0; k < n;) {
        if (n - k == 1 && c.sum.n_pairs == 0) {
            UpdateArgs a{};
            static_cast<UpdateConsts &>(a) = c;
            a.p = segs[k].p;
            a.m = segs[k].m;
            a.v = segs[k].v;
            a.pb = segs[k].pb;
            for (int r = 0; r < R && !CACHED; ++r) a.g[r] = segs[k].g[r];
            a.gbar = segs[k].gbar;
            a.n = segs[k].n;
            a.stride = update_blocks(a.n) * kUpdateThreads;
            return update_r<R>(a, update_blocks(a.n), lds_pad, s);
        }
        SegTable<R> t{};
        int64_t blocks = 0;
        const int done = fill_table<R>(t, segs + k, n - k, CACHED, sdprt::launch_blocks(kUpdateThreads), update_blocks,
                                       &blocks);
        // a call small enough to fold keeps its lines too
        const bool fold = c.sum.n_pairs > 0;
        auto kernel = fold     ? k_update_segments<R, CACHED, true, true>
                      : c.keep ? k_update_segments<R, CACHED, false, true>
                               : k_update_segments<R, CACHED, false, false>;
        hipLaunchKernelGGL(kernel, dim3((uint32_t)blocks), dim3(kUpdateThreads), fold ? 0 : segments_lds_pad, s, t, c);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        k += done;
    }
    return hipSuccess;
}

template <int R>
hipError_t pattern_r(const UpdateArgs &a, int64_t blocks, int lds_pad, hipStream_t s) {
    if (a.gbar)
        hipLaunchKernelGGL((k_update_pattern<1, true>), dim3((uint32_t)blocks), dim3(kUpdateThreads), lds_pad, s, a);
    else
        hipLaunchKernelGGL((k_update_pattern<R, false>), dim3((uint32_t)blocks), dim3(kUpdateThreads), lds_pad, s, a);
    return hipGetLastError();
}

template <int R>
hipError_t norm_pattern_r(const NormArgs &a, int store_lds_pad, hipStream_t s) {
    const int64_t blocks = cdiv(a.n, kTile) * norm_pairs_per_tile(R, true);
    hipLaunchKernelGGL((k_norm_pattern<R>), dim3((uint32_t)blocks), dim3(NormShape<R, true>::kThreads), store_lds_pad, s, a);
    return hipGetLastError();
}

template <int R>
hipError_t gbar_r(const GbarArgs &a, int64_t blocks, hipStream_t s) {
    if (a.bf16)
        hipLaunchKernelGGL((k_gbar_out<R, true>), dim3((uint32_t)blocks), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL((k_gbar_out<R, false>), dim3((uint32_t)blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

#define SDP_FOR_EACH_R(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16)

hipError_t launch_norm_partials(int R, const NormArgs &a, int store_lds_pad, hipStream_t s) {
    switch (R) {
#define CASE(r) case r: return norm_r<r>(a, store_lds_pad, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_norm_segments(int R, const Segment *segs, int n, double *partials, NormState *ns, int keep,
                                int store_lds_pad, hipStream_t s) {
    switch (R) {
#define CASE(r) case r: return norm_segments_r<r>(segs, n, partials, ns, keep, store_lds_pad, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_norm_segments_host(int R, const Segment *segs, int n, double *partials, NormState *ns,
                                     hipStream_t s) {
    switch (R) {
#define CASE(r) case r: return norm_segments_host_r<r>(segs, n, partials, ns, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_update_host(int R, const UpdateArgs &a, hipStream_t s) {
    switch (R) {
#define CASE(r) case r: return update_host_r<r>(a, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_update_segments(int R, const Segment *segs, int n, const UpdateConsts &c, int lds_pad,
                                  int segments_lds_pad, hipStream_t s) {
    if (segs[0].gbar) return update_segments_r<1, true>(segs, n, c, lds_pad, segments_lds_pad, s);
    switch (R) {
#define CASE(r) case r: return update_segments_r<r, false>(segs, n, c, lds_pad, segments_lds_pad, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_norm_finalize(const NormSum &sum, double *merged, hipStream_t s) {
    if (sum.n_pairs < 1) return hipErrorInvalidValue;
    const int64_t run = cdiv(cdiv(sum.n_pairs, kMergeRun), kMaxMergeBlocks) * kMergeRun;
    const int64_t blocks = cdiv(sum.n_pairs, run);
    if (blocks > 1 && !merged) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_norm_finalize, dim3((uint32_t)blocks), dim3(kFinalizeThreads), 0, s, sum, run, merged);
    return hipGetLastError();
}

hipError_t launch_update(int R, UpdateArgs a, int max_blocks, int lds_pad, hipStream_t s) {
    int64_t blocks = update_blocks(a.n);
    if (max_blocks > 0 && blocks > max_blocks) blocks = max_blocks;
    a.stride = blocks * kUpdateThreads;
    switch (R) {
#define CASE(r) case r: return update_r<r>(a, blocks, lds_pad, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_update_pattern(int R, const UpdateArgs &a, int lds_pad, hipStream_t s) {
    int64_t blocks = cdiv(a.n / kUpdVec, kUpdateThreads);
    if (blocks < 1) blocks = 1;
    switch (R) {
#define CASE(r) case r: return pattern_r<r>(a, blocks, lds_pad, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_norm_pattern(int R, const NormArgs &a, int store_lds_pad, hipStream_t s) {
    switch (R) {
#define CASE(r) case r: return norm_pattern_r<r>(a, store_lds_pad, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gbar_out(int R, const GbarArgs &a, int max_blocks, hipStream_t s) {
    int64_t blocks = cdiv(a.n / (a.bf16 ? 8 : 4), 256);
    if (blocks < 1) blocks = 1;
    if (blocks > max_blocks) blocks = max_blocks;
    switch (R) {
#define CASE(r) case r: return gbar_r<r>(a, blocks, s);
        SDP_FOR_EACH_R(CASE)
#undef CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_cast_bf16(const float *src, uint16_t *dst, int64_t n, hipStream_t s) {
    int64_t blocks = cdiv(n / 4, 256);
    if (blocks < 1) blocks = 1;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_cast_bf16, dim3((uint32_t)blocks), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

hipError_t launch_copy16(void *dst, const void *src, int64_t n16, int max_blocks, hipStream_t s) {
    int64_t blocks = cdiv(n16, 256);
    if (blocks < 1) blocks = 1;
    if (max_blocks > 0 && blocks > max_blocks) blocks = max_blocks;
    hipLaunchKernelGGL(k_copy16, dim3((uint32_t)blocks), dim3(256), 0, s, (uint4 *)dst,
                       (const uint4 *)src, n16);
    return hipGetLastError();
}

hipError_t launch_fill_u32(void *dst, int64_t n_words, uint32_t value, hipStream_t s) {
    int64_t blocks = cdiv(n_words / 4, 256);
    if (blocks < 1) blocks = 1;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)blocks), dim3(256), 0, s, (uint32_t *)dst, n_words, value);
    return hipGetLastError();
}

}  // namespace sdp
