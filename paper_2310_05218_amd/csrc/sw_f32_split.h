// fp32 operands for the bf16 matrix instructions: every fp32 value is the sum of three bf16 values
//     v = h + m + l,   h = bf16(v), m = bf16(v - h), l = v - h - m      (rounded to nearest even; the sum is exact),
// and a product is taken as   lh + hl + mm + mh + hm + hh,   six products of eight-bit significands that are exact in the
// fp32 accumulators.  What is left out (ml, lm, ll) is up to 2^-24.0 of the product, as much as an fp32 rounding (both operands
// 1 + 2^-8 - 2^-17; over random pairs 2^-27.5 in the mean square, above 2^-26 for 2.7 % of them).  A sum of a single product is off by
// up to 1.0e-7 of it where an fp32 instruction gives 6e-8 (1.6e-7 in 1 x 1 layers, whose six products share an accumulator), and where
// many equal operands give the left-out parts one sign they are still 2^-24 of the result.
//
// Why: v_mfma_f32_32x32x16_bf16 performs 8 times the multiply-adds of v_mfma_f32_32x32x2_f32 in half its time (per K step of
// 16: 32 cycles against 8 x 64), so six of them still take 0.375 of the fp32 instruction's time; and an accumulator is rounded
// 6 / 16 instead of 1 / 2 times per product.  Against 64-bit sums of N(0,1) data (rel: 2-norm of the error over 2-norm of the
// result), fp32 instruction -> six bf16 ones: 144 products 2.15e-7 -> 1.74e-7, 576: 4.34e-7 -> 3.61e-7, 2304: 8.60e-7 -> 7.42e-7,
// 4608: 1.21e-6 -> 1.07e-6; all products positive, 576: 3.71e-7 -> 2.78e-7; magnitudes spread over 2^40, 576: 3.27e-7 -> 3.21e-7.
// In the layers (the kernels of before -> now): 3 x 3 over 512 channels, N(0,1) 5.8e-7 -> 2.2e-7, all operands 1/3 1.2e-5 -> 5.7e-8;
// 1 x 1 over 256, N(0,1) 2.9e-7 -> 2.4e-7, operands within 2e-7 of 1 + 2^-8 - 2^-17 8.6e-8 -> 1.3e-7; 7 x 7 over 3, N(0,1) 2.1e-7 -> 6.9e-8.
//
// Range.  A value is split after a factor of 2^24, and a sum of products leaves with a factor of 2^-48 (split_unscale).  Scaled so,
// every part of every fp32 value, denormal ones included, is a normal bf16 value or zero (the last bit of the smallest value is
// 2^-149, of its part 2^-125) and no product a result can show underflows: small values need no test and cost nothing.  The
// other end pays: a value from about 2^104 up, an infinity or a NaN has a NaN for a part, a sum from 2^80 up overflows, and either
// leaves no finite number in the accumulators that meet it.  The blocks of those, and only those, are computed again on the fp32
// instruction (multiply_f32), and the lanes concerned (a pixel's sixteen channels) take that result: which outputs these are follows
// from the operands alone.  Cost (us, 32 images; without / one NaN in x / one in w / x all NaN): 3 x 3, 64 -> 64 at 56 x 56 53 / 138 /
// 185 / 293, 7 x 7 stride 2, 3 -> 64 at 224 x 224 58 / 67 / 241 / 304, 1 x 1, 256 -> 64 at 56 x 56 31 / 69 / 128 / 229, one
// image of 256 -> 256 at 14 x 14 18 / 161 / 161 / 162; a value of 1e-38 in either place costs nothing.
#pragma once

#include "swconv_internal.h"

namespace swconv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float splitx16 __attribute__((ext_vector_type(16)));

struct Split8 {
    bf16x8 h, m, l;
};

constexpr int kSplitExponent = 24;
constexpr float kSplitUnscale = 0x1p-48f;

// Splits eight values.
// In pairs and in stages: v_cvt_pk_bf16_f32 takes two values and nothing waits for the instruction before it (25 ticks a
// value; written value by value the compiler converts each one alone and once more to pack it, three times slower).
__device__ __forceinline__ Split8 split_f32(const float (&v)[8])
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
    for (int j = 0; j < 8; ++j) e[j] = __builtin_amdgcn_ldexpf(v[j], kSplitExponent);     // (a multiplication moves to where the value is loaded)
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = pack(e[2 * j], e[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        e[2 * j] -= even(h[j]);
        e[2 * j + 1] -= odd(h[j]);
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
    return Split8{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

// Whether an accumulator holds an infinity or a NaN.  (In integer maxima: as sixteen comparisons the compiler gathers them bit by bit.)
__device__ __forceinline__ bool split_overflow(const splitx16& acc)
{
    unsigned hi = 0;
#pragma unroll
    for (int v = 0; v < 16; ++v) hi = max(hi, __float_as_uint(acc[v]) << 1);
    return hi >= 0x7f800000u << 1;
}
__device__ __forceinline__ void split_unscale(splitx16& acc)
{
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] *= kSplitUnscale;
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

// A wavefront's block of 32 output channels x 32 pixels on the fp32 matrix instruction, its operands straight from memory: for
// blocks with accumulators that hold no finite number, after their stores (registers), by all lanes of the wavefront.  Lane half kk
// takes a half of a filter's `per` taps; row: the filter of lane lj (beyond the last: the last, and not stored); at(in): the next
// input of the lane's pixel, zero unless `in`; U: loads in flight per operand.  Registers as those of the accumulators it replaces.
// The empty statements here keep the compiler from computing any of this where every launch passes.
template <int U, class Inputs>
__device__ __forceinline__ splitx16 multiply_f32(const float* __restrict__ w, int per, int row, int C_out, int kk, Inputs at)
{
    asm volatile("" : "+v"(per), "+v"(row));
    const int half = (per + 1) >> 1, count = kk ? per - half : half;
    const float* wp = w + (int64_t)min(row, C_out - 1) * per + kk * half;
    splitx16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll 1
    for (int t = 0; t < __builtin_amdgcn_readfirstlane(half); t += U) {
        float a[U], b[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const bool in = t + j < count;
            a[j] = wp[in ? t + j : 0];
            b[j] = at(in);
            if (!in) a[j] = 0.f;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < U; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], acc, 0, 0, 0);
    }
    return acc;
}
__device__ __forceinline__ void store_outputs(const splitx16& acc, float* yp, int HoWo, int co, int C_out, const Epilogue& ep)
{
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int c = 8 * (v >> 2) + (v & 3);
        if (co + c < C_out) yp[(int64_t)c * HoWo] = apply_epilogue(acc[v], co + c, ep);
    }
}

// The inputs of output (n, oh, ow) for multiply_f32, from tap `first` on; zeros where the filter lies over the padding.
// (x: less than 2 GiB)
struct ConvInputs {
    __amdgpu_buffer_rsrc_t xr;
    int H, W, R, S, dil, top, left, r, s;
    unsigned plane;                                     // byte offset of the current channel's plane
    __device__ __forceinline__ ConvInputs(__amdgpu_buffer_rsrc_t xr, int C_in, int H, int W, int R, int S, int stride, int pad, int dil, int n, int oh,
                                          int ow, int first)
        : xr(xr), H(H), W(W), R(R), S(S), dil(dil), top(oh * stride - pad), left(ow * stride - pad)
    {
        int taps = R * S, cols = S;
        asm volatile("" : "+v"(taps), "+v"(cols), "+v"(n), "+v"(first));
        const int ci = first / taps, tap = first - ci * taps;
        r = tap / cols;
        s = tap - r * cols;
        plane = (unsigned)(n * C_in + ci) * (unsigned)(H * W) * 4u;
    }
    __device__ __forceinline__ float operator()(bool in)
    {
        const int gr = top + r * dil, gc = left + s * dil;
        // (without branches, which would keep the loads apart)
        const bool inside = in & ((unsigned)gr < (unsigned)H) & ((unsigned)gc < (unsigned)W);
        const unsigned off = inside ? plane + (unsigned)(gr * W + gc) * 4u : 0x80000000u;
        const bool row_end = s + 1 == S, plane_end = row_end & (r + 1 == R);
        s = row_end ? 0 : s + 1;
        r = plane_end ? 0 : row_end ? r + 1 : r;
        plane += plane_end ? (unsigned)(H * W) * 4u : 0u;
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, off, 0, 0));
    }
};

// ... and of one tap: `step` values apart (once they have ended, the last one is read again and not used).
struct ColumnInputs {
    const float* p;
    int step;
    __device__ __forceinline__ float operator()(bool in)
    {
        const float v = *(in ? p : p - step);
        p += in ? step : 0;
        return in ? v : 0.f;
    }
};

}  // namespace swconv
