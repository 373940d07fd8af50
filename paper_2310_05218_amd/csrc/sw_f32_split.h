// fp32 operands for the bf16 matrix instructions: every fp32 value is the sum of three bf16 values
//     v = h + m + l,   h = bf16(v), m = bf16(v - h), l = v - h - m      (rounded to nearest even; the sum is exact),
// and a product is taken as   lh + hl + mm + mh + hm + hh,   six products of eight-bit significands that are exact in the
// fp32 accumulators.  What is left out (ml, lm, ll) is at most 2^-26 of the product, below the rounding of one fp32 addition.
//
// Why: v_mfma_f32_32x32x16_bf16 performs 16 times the multiply-adds of v_mfma_f32_32x32x2_f32 in half its time per K step of
// 16 (32 cycles against 8 x 64), so six of them still take 0.375 of the fp32 instruction's time; and an accumulator is rounded
// 6 / 16 instead of 1 / 2 times per product.  Against 64-bit sums of N(0,1) data (rel: 2-norm of the error over 2-norm of the
// result), fp32 instruction -> six bf16 ones: 144 products 2.15e-7 -> 1.74e-7, 576: 4.34e-7 -> 3.61e-7, 2304: 8.60e-7 -> 7.42e-7,
// 4608: 1.21e-6 -> 1.07e-6; all products positive, 576: 3.71e-7 -> 2.78e-7; magnitudes spread over 2^40, 576: 3.27e-7 -> 3.21e-7.
//
// The sum h + m + l is exact for every finite value from about 2^-102 up to the largest bf16.  An infinity, a NaN or a larger
// value has a NaN for m or l, which makes a NaN of every accumulator it meets; values below 2^-102 (whose l would leave the
// bf16 range) are reported by split_f32 through `tiny`.  Kernels compute what either can reach by plain fp32 multiply-adds.
#pragma once

#include "swconv_internal.h"

namespace swconv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float splitx16 __attribute__((ext_vector_type(16)));

struct Split8 {
    bf16x8 h, m, l;
};

// Splits eight values; `tiny` becomes the smallest of (bits of |v|) * 2 - 1 (a zero counts as the largest).
// In pairs and in stages: v_cvt_pk_bf16_f32 takes two values and nothing waits for the instruction before it (25 ticks a
// value; written value by value the compiler converts each one alone and once more to pack it, three times slower).
__device__ __forceinline__ Split8 split_f32(const float (&v)[8], unsigned& tiny)
{
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
    auto pack = [](float a, float b) __attribute__((always_inline)) {
        const floatx2 p = {a, b};
        return __builtin_bit_cast(unsigned, __builtin_convertvector(p, bf16x2));
    };
    auto even = [](unsigned p) __attribute__((always_inline)) { return __uint_as_float(p << 16); };
    auto odd = [](unsigned p) __attribute__((always_inline)) { return __uint_as_float(p & 0xffff0000u); };
    uintx4 h, m, l;
    float e[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = pack(v[2 * j], v[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        e[2 * j] = v[2 * j] - even(h[j]);
        e[2 * j + 1] = v[2 * j + 1] - odd(h[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) m[j] = pack(e[2 * j], e[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        e[2 * j] -= even(m[j]);
        e[2 * j + 1] -= odd(m[j]);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) l[j] = pack(e[2 * j], e[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 8; ++j) tiny = min(tiny, (__float_as_uint(v[j]) << 1) - 1u);
    return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
constexpr unsigned kTinyBits = 0x0c800000u << 1;        // 2^-102, as `tiny` counts

// Accumulators that may have lost something the operands had: not finite, or so small (below 2^-100, but not zero) that
// partial products underflowed.  (In integer minima and maxima: as sixteen comparisons the compiler gathers them bit by bit.)
__device__ __forceinline__ bool split_suspect(const splitx16& acc)
{
    unsigned hi = 0, lo = ~0u;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const unsigned a = __float_as_uint(acc[v]) << 1;
        hi = max(hi, a);
        lo = min(lo, a - 1u);
    }
    return hi >= 0x7f800000u << 1 || lo < (0x0d800000u << 1) - 1u;
}

// Stores a block's 32 output channels x 32 pixels: register v of a lane is output channel co + 8 (v / 4) + v % 4 of its pixel
// (co: the lane's first channel, yp: its place), channels HoWo floats apart; nontemporal, because a launch's last lines would
// otherwise wait in L2 for its end.  Whole blocks without a test per value: sixteen of them, each with the tests of the
// epilogue, cost more than the stores.
__device__ __forceinline__ void store_block(splitx16 acc, float* yp, int HoWo, int co, int C_out, bool whole, const Epilogue& ep)
{
    if (whole) {
        if (ep.bias) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] += ep.bias[co + 8 * (v >> 2) + (v & 3)];
        }
        if (ep.relu) {
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = fmaxf(acc[v], 0.f);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) __builtin_nontemporal_store(acc[v], yp + (int64_t)(8 * (v >> 2) + (v & 3)) * HoWo);
    } else {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int c = 8 * (v >> 2) + (v & 3);
            if (co + c < C_out) __builtin_nontemporal_store(apply_epilogue(acc[v], co + c, ep), yp + (int64_t)c * HoWo);
        }
    }
}

// One output by plain fp32 multiply-adds, taps in the padding as zeros: what an accumulator that is no use is replaced by.
__device__ inline float conv_output_f32(const float* __restrict__ x, const float* __restrict__ w, int C_in, int H, int W, int R, int S,
                                        int stride, int pad, int dil, int n, int co, int oh, int ow)
{
    float acc = 0.f;
    const float* wp = w + (int64_t)co * C_in * R * S;
#pragma unroll 1
    for (int ci = 0; ci < C_in; ++ci) {
        const float* xp = x + ((int64_t)n * C_in + ci) * H * W;
#pragma unroll 1
        for (int r = 0; r < R; ++r)
#pragma unroll 1
            for (int s = 0; s < S; ++s, ++wp) {
                const int gr = oh * stride - pad + r * dil, gc = ow * stride - pad + s * dil;
                const bool in = gr >= 0 && gr < H && gc >= 0 && gc < W;
                acc = fmaf(in ? xp[(int64_t)gr * W + gc] : 0.f, *wp, acc);
            }
    }
    return acc;
}

}  // namespace swconv
