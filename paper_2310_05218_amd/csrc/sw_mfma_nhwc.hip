// Multi-channel convolution on channel-last tensors, fp32, bf16 and IEEE half, on the matrix cores: any filter extent,
// stride, padding and dilation (paper, section 3: the taps as small matrix products; section 1.1: reduced
// precision applied to the same sliding formulation).
//
//   x [N, H, W, C_in]     w [C_out, R, S, C_in]     y [N, H_out, W_out, C_out]
//   fp32: fp32 everywhere, v_mfma_f32_32x32x2_f32.
//   bf16: x, w and y are bf16 bit patterns, products and sums are fp32 (v_mfma_f32_32x32x16_bf16: a bf16 product
//         is exact in fp32), one rounding of the finished sum (+ bias, rectifier) to bf16, nearest even.
//   half: the same with v_mfma_f32_32x32x16_f16 (a product of two halves is exact in fp32 as well) and one rounding
//         to half precision, nearest even, overflow to infinity, denormals kept.
//
// With the channel as the fastest axis of both tensors the K operand of a matrix instruction is 16 consecutive
// bytes of memory per lane (four fp32 channels = the operands of four K steps, or eight bf16 channels = one), so
// nothing is transposed on the way: the rows of the input a band of outputs touches and the filters of 64 output
// channels go to LDS with plain 16-byte loads, a chunk of CB bytes per pixel at a time (all loads of a chunk are
// issued before the first LDS write: one memory round trip), and every tap (r, s) contributes W_rs[co, ci] times
// the window shifted by (r, s) * dilation: the shift is an address offset, no column matrix exists.
//
// Workgroup = 4 wavefronts = 64 output channels x a band of TH output rows of one image, taken as up to 8 blocks
// of 32 consecutive output pixels (row-major: each lane computes its own pixel's window address).  A = pixels,
// B = filters: a lane of the result holds one output channel for 16 pixels, so a store instruction writes runs of
// 32 consecutive channels, the fastest axis of the output.  LDS pitches: a pixel takes CB + 16 bytes, an output
// channel's filters R*S*CB + 16 (+ what makes that 16 modulo 128).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "swconv_internal.h"

namespace swconv {

namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

constexpr int kMaxBlocks = 8;          // 32-pixel blocks per workgroup
constexpr int kBlocksPerWave = 4;      // a wavefront takes every second block of one 32-channel half
constexpr int kLdsBudget = 156 * 1024;
constexpr int kXSlots = 12;            // 16-byte pieces of the window per thread and chunk
constexpr int kWSlots = 24;            // 16-byte pieces of the filters per thread and chunk

struct NhwcFParams {
    Epilogue ep;                       // fp32 bias and rectifier applied in the store
    int H, W, C_out, R, S, stride, pad, dil, Ho, Wo;
    int PB, CB, chunks;                // bytes per pixel (C_in * element size), per pixel and chunk, chunks
    int TH, IH, IWp;                   // output rows per band; window rows and columns in LDS
    int CP, WPITCH;                    // bytes per pixel / per output channel's filters in LDS
    int c16;                           // 16-byte pieces per pixel and chunk
    int wrow16;                        // 16-byte pieces per output channel's filters and chunk (R * S * c16)
    int x_bytes;                       // window bytes in LDS (filters follow)
    FastDiv by_c16, by_IWp, by_wrow16, by_Wo;
};

__device__ __forceinline__ unsigned short bf16_rne(float f)
{
    unsigned u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// the one rounding of a finished value to the tensor's 16-bit format
template <int EK>
__device__ __forceinline__ unsigned short round16(float f)
{
    if constexpr (EK == kElemF16) return __builtin_bit_cast(unsigned short, (_Float16)f);      // v_cvt_f16_f32: nearest even
    else return bf16_rne(f);
}

// a 16-bit element widened to fp32 (exact)
template <int EK>
__device__ __forceinline__ float widen16(unsigned short h)
{
    if constexpr (EK == kElemF16) return (float)__builtin_bit_cast(_Float16, h);
    else return __uint_as_float((unsigned)h << 16);
}

// EK: element format (Elem).  KS: K steps of 32 bytes per tap and chunk (CB / 32): 1, 2 or 4.
template <int EK, int KS>
__global__ __launch_bounds__(256, 1) void mfma_nhwc_kernel(const unsigned char* __restrict__ x,
                                                           const unsigned char* __restrict__ w, void* __restrict__ yv,
                                                           const NhwcFParams P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    unsigned char* lx = smem;                 // [window row][window column][chunk bytes], pitch CP
    unsigned char* lw = smem + P.x_bytes;     // [co][tap][chunk bytes], pitch WPITCH
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int lg = lane >> 5, lj = lane & 31;          // K half; pixel (A) or channel (B, D) inside a block
    const int band = blockIdx.x, n = blockIdx.y, cb = blockIdx.z;
    const int oi0 = band * P.TH;                        // first output row of the band
    const int rows = min(P.TH, P.Ho - oi0);
    const int npix = rows * P.Wo;                       // output pixels of this band
    const int co0 = cb * 64;
    const int RS = P.R * P.S;

    // ---- staging plan (the same for every chunk): window piece = (window pixel, 16-byte piece c of the chunk)
    const int gr0 = oi0 * P.stride - P.pad;             // image row / column of window position (0, 0)
    const int n_x = P.IH * P.IWp * P.c16;
    const unsigned char* xn = x + (int64_t)n * P.H * P.W * P.PB;
    int xsrc[kXSlots], xdst[kXSlots];                   // source byte offset in the image (< 0: zero), LDS byte offset (< 0: none)
#pragma unroll
    for (int u = 0; u < kXSlots; ++u) {
        const int idx = tid + 256 * u;
        const int pix = fast_div(idx, P.by_c16);
        const int c = idx - pix * P.c16;
        const int e = fast_div(pix, P.by_IWp), f = pix - e * P.IWp;
        const int gr = gr0 + e, gc = f - P.pad;
        xdst[u] = idx < n_x ? pix * P.CP + 16 * c : -1;
        xsrc[u] = (idx < n_x && gr >= 0 && gr < P.H && gc >= 0 && gc < P.W) ? (gr * P.W + gc) * P.PB + 16 * c : -1;
    }
    // filter piece = (output channel, tap, 16-byte piece c of the chunk)
    const int n_w = 64 * P.wrow16;
    const unsigned char* wb = w + (int64_t)co0 * RS * P.PB;

    // ---- this wavefront: channel half wn, pixel blocks wp, wp + 2, wp + 4, wp + 6 ----
    const int wn = wave & 1, wp = wave >> 1;
    const int nblocks = (npix + 31) >> 5;
    int aoff[kBlocksPerWave];                           // byte offset in lx of the lane's pixel, tap (0, 0)
#pragma unroll
    for (int b = 0; b < kBlocksPerWave; ++b) {
        int p = 32 * (wp + 2 * b) + lj;
        if (p > npix - 1) p = npix - 1;                 // lanes past the band read a valid pixel, store nothing
        const int oi = fast_div(p, P.by_Wo), oj = p - oi * P.Wo;
        aoff[b] = ((oi * P.stride) * P.IWp + oj * P.stride) * P.CP + 16 * lg;
    }
    const unsigned char* bsrc = lw + (32 * wn + lj) * P.WPITCH + 16 * lg;
    floatx16 acc[kBlocksPerWave];
#pragma unroll
    for (int b = 0; b < kBlocksPerWave; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[b][v] = 0.f;

    struct Ops {
        intx4 bq[KS];
        intx4 aq[KS][kBlocksPerWave];
    };
    auto load_ops = [&](Ops& o, int tap_x, int tap_w) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            o.bq[k] = *reinterpret_cast<const intx4*>(bsrc + tap_w + 32 * k);
#pragma unroll
            for (int b = 0; b < kBlocksPerWave; ++b)
                o.aq[k][b] = *reinterpret_cast<const intx4*>(lx + aoff[b] + tap_x + 32 * k);
        }
    };
    auto multiply = [&](const Ops& o) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < KS; ++k)
#pragma unroll
            for (int b = 0; b < kBlocksPerWave; ++b)
                if (wp + 2 * b < nblocks) {             // (wave-uniform)
                    if constexpr (EK == kElemF16) {
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, o.aq[k][b]),
                                                                        __builtin_bit_cast(halfx8, o.bq[k]), acc[b], 0, 0, 0);
                    } else if constexpr (EK == kElemBF16) {
                        acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o.aq[k][b]),
                                                                         __builtin_bit_cast(bf16x8, o.bq[k]), acc[b], 0, 0, 0);
                    } else {
                        const floatx4 af = __builtin_bit_cast(floatx4, o.aq[k][b]), bf = __builtin_bit_cast(floatx4, o.bq[k]);
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[t], bf[t], acc[b], 0, 0, 0);
                    }
                }
    };

    for (int ch = 0; ch < P.chunks; ++ch) {
        // ---- global -> registers -> LDS: every piece of the chunk before any LDS write
        const int cb0 = ch * P.CB;
        intx4 xv[kXSlots];
#pragma unroll
        for (int u = 0; u < kXSlots; ++u) {
            xv[u] = intx4{0, 0, 0, 0};
            if (xsrc[u] >= 0) xv[u] = *reinterpret_cast<const intx4*>(xn + xsrc[u] + cb0);
        }
        if (ch > 0) __syncthreads();                    // everybody has finished the multiplications of the chunk before
#pragma unroll
        for (int u = 0; u < kXSlots; ++u)
            if (xdst[u] >= 0) *reinterpret_cast<intx4*>(lx + xdst[u]) = xv[u];
        // the filters in rounds of kWSlots pieces per thread (one round for up to 96 pieces per output channel)
        for (int base = 0; base < n_w; base += 256 * kWSlots) {
            intx4 wv[kWSlots];
            int wdst[kWSlots];
#pragma unroll
            for (int u = 0; u < kWSlots; ++u) {
                const int idx = base + tid + 256 * u;
                const int co = fast_div(idx, P.by_wrow16);
                const int q = idx - co * P.wrow16;
                const int tap = fast_div(q, P.by_c16), c = q - tap * P.c16;
                wdst[u] = idx < n_w ? co * P.WPITCH + tap * P.CB + 16 * c : -1;
                wv[u] = intx4{0, 0, 0, 0};              // channels beyond C_out: zero filters
                if (idx < n_w && co0 + co < P.C_out)
                    wv[u] = *reinterpret_cast<const intx4*>(wb + (co * RS + tap) * P.PB + 16 * c + cb0);
            }
#pragma unroll
            for (int u = 0; u < kWSlots; ++u)
                if (wdst[u] >= 0) *reinterpret_cast<intx4*>(lw + wdst[u]) = wv[u];
        }
        __syncthreads();

        // ---- every tap: the operands of the next tap are on their way from LDS while this one multiplies
        int tap_x = 0, tap_w = 0, s = 0;
        auto next_tap = [&]() __attribute__((always_inline)) {
            tap_w += P.CB;
            tap_x += P.dil * P.CP;
            if (++s == P.S) { s = 0; tap_x += P.dil * (P.IWp - P.S) * P.CP; }
        };
        Ops o0, o1;
        load_ops(o0, tap_x, tap_w);
        int tap = 0;
#pragma unroll 1
        for (; tap + 2 <= RS; tap += 2) {
            next_tap();
            load_ops(o1, tap_x, tap_w);
            __builtin_amdgcn_sched_barrier(0);
            multiply(o0);
            __builtin_amdgcn_sched_barrier(0);
            if (tap + 2 < RS) {
                next_tap();
                load_ops(o0, tap_x, tap_w);
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(o1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (tap < RS) multiply(o0);                     // odd tap count: the last tap is already in o0
    }

    // ---- store: register v of a lane is pixel 8*(v/4) + 4*lg + v%4 of the block, channel lj ----
    const int co = co0 + 32 * wn + lj;
    if (co >= P.C_out) return;
    const int64_t pix0 = ((int64_t)n * P.Ho + oi0) * P.Wo;
    const float bias = P.ep.bias ? P.ep.bias[co] : 0.f;
#pragma unroll
    for (int b = 0; b < kBlocksPerWave; ++b) {
        if (wp + 2 * b >= nblocks) break;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int p = 32 * (wp + 2 * b) + 8 * (v >> 2) + 4 * lg + (v & 3);
            float t = acc[b][v];
            if (P.ep.bias) t += bias;
            if (P.ep.relu) t = fmaxf(t, 0.f);
            if (p < npix) {
                if constexpr (EK != kElemF32) static_cast<unsigned short*>(yv)[(pix0 + p) * P.C_out + co] = round16<EK>(t);
                else static_cast<float*>(yv)[(pix0 + p) * P.C_out + co] = t;
            }
        }
    }
}

// One thread per output, any shape: the channel loop runs over contiguous elements of both tensors.
template <int EK>
__global__ __launch_bounds__(256) void direct_nhwc_kernel(const void* __restrict__ xv, const void* __restrict__ wv,
                                                          void* __restrict__ yv, Conv2dShape s, Epilogue ep)
{
    const int64_t total = (int64_t)s.N * s.Ho * s.Wo * s.C_out;
    for (int64_t o = (int64_t)blockIdx.x * 256 + threadIdx.x; o < total; o += (int64_t)gridDim.x * 256) {
        const int co = (int)(o % s.C_out);
        int64_t t = o / s.C_out;
        const int oj = (int)(t % s.Wo);
        t /= s.Wo;
        const int oi = (int)(t % s.Ho);
        const int n = (int)(t / s.Ho);
        float acc = 0.f;
        for (int r = 0; r < s.R; ++r) {
            const int h = oi * s.stride + r * s.dil - s.pad;
            if (h < 0 || h >= s.H) continue;
            for (int q = 0; q < s.S; ++q) {
                const int v = oj * s.stride + q * s.dil - s.pad;
                if (v < 0 || v >= s.W) continue;
                const int64_t xo = (((int64_t)n * s.H + h) * s.W + v) * s.C_in, wo = (((int64_t)co * s.R + r) * s.S + q) * s.C_in;
                if constexpr (EK != kElemF32) {
                    const unsigned short* xp = static_cast<const unsigned short*>(xv) + xo;
                    const unsigned short* wp = static_cast<const unsigned short*>(wv) + wo;
                    for (int ci = 0; ci < s.C_in; ++ci)
                        acc = fmaf(widen16<EK>(xp[ci]), widen16<EK>(wp[ci]), acc);
                } else {
                    const float* xp = static_cast<const float*>(xv) + xo;
                    const float* wp = static_cast<const float*>(wv) + wo;
                    for (int ci = 0; ci < s.C_in; ++ci) acc = fmaf(xp[ci], wp[ci], acc);
                }
            }
        }
        if (ep.bias) acc += ep.bias[co];
        if (ep.relu) acc = fmaxf(acc, 0.f);
        if constexpr (EK != kElemF32) static_cast<unsigned short*>(yv)[o] = round16<EK>(acc);
        else static_cast<float*>(yv)[o] = acc;
    }
}

// Up to four input channels (the first layer of a network): 2 to 8 bytes a pixel are no K step of a matrix instruction.  The filters,
// turned to [tap][channel][output channel], and the input rows under a band of output rows go to LDS as fp32, padding as zeros; a thread
// owns eight consecutive output channels of PX consecutive pixels of a row, so that two 16-byte reads of filters feed 8 PX multiply-adds
// and a wavefront stores whole runs of channels.  The sums run in the order of the one-thread-per-output kernel, to the same bits; that one
// leaves taps in the padding out, which only an infinite or NaN filter value can tell from a product with zero: then the taps are tested.
//
// Measured (us, replayed graphs of ten, 3x3 at stride 2 on three channels, against one thread per output):
// half, 4 x 210 x 198 to 64 channels 74.7 -> 10.3, 4 x 152 x 108 31.1 -> 8.4, 32 x 224 x 224 649 -> 45 (31 TFLOP/s), 7x7 on 8 x 224 x 224
// 901 -> 62; fp32 4 x 152 x 108 33.6 -> 7.7.  Staging without branches, since: half 2 x 104 x 109 8.1 -> 7.1, 1.10 x over 50 layers; reading a tap's
// operands before the products of the one before was 0.96 x, eight values in flight 1.02 x.  Bound by the round trip in front of the barrier and, of small launches, a thread's chain of
// LDS reads and multiply-adds; of large ones by those.
struct FewNhwcParams {
    Epilogue ep;
    int H, W, C_out, R, S, stride, pad, dil, Ho, Wo, TH, bands, IH, pitch;      // pitch: floats of a framed input row
    int octets, slots, groups;          // of output channels, threads with the same octet, groups of four pixels per output row
    FastDiv by_pitch, by_octets, by_groups, by_bands, by_K;
};

template <int EK, int CI, int PX>
__global__ __launch_bounds__(256) void few_channels_nhwc_kernel(const void* __restrict__ xv, const void* __restrict__ wv, void* __restrict__ yv,
                                                                const FewNhwcParams P)
{
    extern __shared__ __attribute__((aligned(16))) float few_lds[];
    const int tid = threadIdx.x, taps = P.R * P.S, K = taps * CI;
    const int wp = P.C_out + 4;                     // (consecutive taps four banks apart: they arrive together)
    float* ws = few_lds;                            // [K][wp]
    float* xs = few_lds + K * wp;                   // [IH][pitch]
    const int n = fast_div(blockIdx.x, P.by_bands), o0 = (blockIdx.x - n * P.bands) * P.TH;
    auto value = [](const void* p, int64_t i) __attribute__((always_inline)) {
        if constexpr (EK != kElemF32) return widen16<EK>(static_cast<const unsigned short*>(p)[i]);
        else return static_cast<const float*>(p)[i];
    };
    const int slot = fast_div(tid, P.by_octets), co = 8 * (tid - slot * P.octets);
    float bias[8] = {};
    if (P.ep.bias && slot < P.slots) {
#pragma unroll
        for (int c = 0; c < 8; ++c) bias[c] = P.ep.bias[co + c];
    }
    // four input values and four filter values in flight per thread
    const int64_t first = (int64_t)n * P.H * P.W * CI;
    const int cells = P.IH * P.pitch, rowlen = P.W * CI, filters = K * P.C_out;
    bool beyond = false;
    for (int base = tid; base < max(cells, filters); base += 4 * 256) {
        float v[4], f[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + 256 * u, r = fast_div(i, P.by_pitch), e = i - r * P.pitch - P.pad * CI, h = o0 * P.stride - P.pad + r;
            const bool in = i < cells && h >= 0 && h < P.H && e >= 0 && e < rowlen;
            if constexpr (EK == kElemF32) {
                v[u] = in ? value(xv, first + (int64_t)h * rowlen + e) : 0.f;
                f[u] = i < filters ? value(wv, i) : 0.f;
            } else {
                // (loads of the first value in place of branches around them, which would be waited for one by one: their halves of a register are
                // widened behind each.  fp32 values need nothing of the kind and were 0.91 to 1.04, 0.99 on the average, as fast so)
                const float vx = value(xv, first + (in ? (int64_t)h * rowlen + e : 0)), vw = value(wv, i < filters ? i : 0);
                v[u] = in ? vx : 0.f;
                f[u] = vw;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + 256 * u;
            if (i < cells) xs[i] = v[u];
            if (i < filters) {
                const int c = fast_div(i, P.by_K);
                ws[(i - c * K) * wp + c] = f[u];
                beyond |= !(fabsf(f[u]) < INFINITY);
            }
        }
    }
    const bool strict = __syncthreads_or(beyond) != 0;
    if (slot >= P.slots) return;
    const int items = min(P.TH, P.Ho - o0) * P.groups;
    for (int it = slot; it < items; it += P.slots) {
        const int tr = fast_div(it, P.by_groups), j0 = PX * (it - tr * P.groups), oi = o0 + tr;
        float acc[PX][8] = {};
        int at[PX];
#pragma unroll
        for (int j = 0; j < PX; ++j) at[j] = tr * P.stride * P.pitch + min(j0 + j, P.Wo - 1) * P.stride * CI;
        auto sum = [&](auto tested) __attribute__((always_inline)) {
            int k = 0;
#pragma unroll 1
            for (int r = 0; r < P.R; ++r)
#pragma unroll 1
                for (int q = 0; q < P.S; ++q) {
                    const float* xp = xs + r * P.dil * P.pitch + q * P.dil * CI;
                    bool in[PX];
                    if constexpr (tested.value) {
                        const int h = oi * P.stride + r * P.dil - P.pad;
#pragma unroll
                        for (int j = 0; j < PX; ++j) {
                            const int v = (j0 + j) * P.stride + q * P.dil - P.pad;
                            in[j] = h >= 0 && h < P.H && v >= 0 && v < P.W;
                        }
                    }
#pragma unroll
                    for (int ci = 0; ci < CI; ++ci, ++k) {
                        const floatx4 a = *reinterpret_cast<const floatx4*>(ws + k * wp + co), b = *reinterpret_cast<const floatx4*>(ws + k * wp + co + 4);
                        const float f[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
                        for (int j = 0; j < PX; ++j) {
                            const float v = xp[at[j] + ci];
#pragma unroll
                            for (int c = 0; c < 8; ++c) {
                                const float s = fmaf(v, f[c], acc[j][c]);
                                if constexpr (tested.value) acc[j][c] = in[j] ? s : acc[j][c];
                                else acc[j][c] = s;
                            }
                        }
                    }
                }
        };
        if (strict) sum(std::true_type{});
        else sum(std::false_type{});
#pragma unroll
        for (int j = 0; j < PX; ++j) {
            if (j0 + j >= P.Wo) break;
            const int64_t o = (((int64_t)n * P.Ho + oi) * P.Wo + j0 + j) * P.C_out + co;
            float t[8];
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                t[c] = acc[j][c];
                if (P.ep.bias) t[c] += bias[c];
                if (P.ep.relu) t[c] = fmaxf(t[c], 0.f);
            }
            if constexpr (EK != kElemF32) {
                intx4 v;
#pragma unroll
                for (int c = 0; c < 4; ++c) v[c] = (int)(round16<EK>(t[2 * c]) | (unsigned)round16<EK>(t[2 * c + 1]) << 16);
                *reinterpret_cast<intx4*>(static_cast<unsigned short*>(yv) + o) = v;
            } else {
                *reinterpret_cast<floatx4*>(static_cast<float*>(yv) + o) = floatx4{t[0], t[1], t[2], t[3]};
                *reinterpret_cast<floatx4*>(static_cast<float*>(yv) + o + 4) = floatx4{t[4], t[5], t[6], t[7]};
            }
        }
    }
}

// us of a launch with filters and rows in LDS, and of one with a thread per output, fitted to 11151 drawn layers of both (1 to 32 images, 1 to 2000
// rows and columns, 1 to 121 taps, strides 1 to 16, 8 to 256 output channels; both within 18 and 19 % of what was measured, 2-norm).  The
// first pays for a workgroup's filters a thousand at a time and for a thread's chain of products, however few outputs share them.
double few_nhwc_us(const FewNhwcParams& P, int PX, int64_t K, int64_t grid, size_t lds)
{
    const double fill = (double)std::max<int64_t>((int64_t)P.IH * P.pitch, K * P.C_out);
    const double chain = (double)K * ((P.TH * P.groups + P.slots - 1) / P.slots);
    const double at_once = 256.0 * std::max<int64_t>(1, std::min<int64_t>(160 * 1024 / (int64_t)(lds + 256), PX == 4 ? 4 : 8));
    return 3.2 + std::ceil(grid / at_once) * (0.76 * std::ceil(fill / 1024) + (PX == 4 ? 0.084 : 0.033) * chain) +
           std::ceil(grid / 256.0) * (1.3e-5 * fill + (PX == 4 ? 0.044 : 0.0115) * chain + 0.42);
}
double one_per_output_nhwc_us(const Conv2dShape& s)
{
    // (taps outside the image cost a test)
    const double taps = (double)std::min(s.R, (s.H + s.dil - 1) / s.dil) * std::min(s.S, (s.W + s.dil - 1) / s.dil), K = taps * s.C_in;
    return 2.7 + 0.072 * K + 0.059 * s.R * s.S + 0.88e-6 * ((double)s.N * s.Ho * s.Wo * s.C_out) * (K + 1.8);
}

struct FewNhwcPlan {
    FewNhwcParams P;
    unsigned grid;
    size_t lds;
    int PX;
    bool ok;
};

FewNhwcPlan plan_few_nhwc(const Conv2dShape& s, const void* y)
{
    FewNhwcPlan a{};
    FewNhwcParams& P = a.P;
    if (s.C_in > 4 || s.C_out % 8 != 0 || s.C_out > 256 || reinterpret_cast<uintptr_t>(y) % 16 != 0) return a;
    const int64_t pitch = ((int64_t)(s.Wo - 1) * s.stride + (int64_t)(s.S - 1) * s.dil + 1) * s.C_in;
    const int64_t filters = (int64_t)s.R * s.S * s.C_in * (s.C_out + 4), span = (int64_t)(s.R - 1) * s.dil + 1;
    constexpr int64_t kFloats = 16 * 1024;          // 64 KB beside the 256 bytes of __syncthreads_or: two workgroups per CU
    if (filters + span * pitch > kFloats) return a;
    P.octets = s.C_out / 8;
    P.slots = 256 / P.octets;
    // four pixels a thread for long sums (7x7 on three channels 28.3 us against 36.5 with one, 8 images 62 against 78) and where a row is
    // more than three turns of the workgroup at one (105 x 99 outputs of 64 channels 10.3 against 12.0), one otherwise (76 x 54 8.4 against
    // 9.2, 32 x 32 of one image 5.4 against 7.9: half the latency of a thread's chain)
    a.PX = s.R * s.S * s.C_in >= 64 || s.Wo > 3 * P.slots ? 4 : 1;
    P.groups = (s.Wo + a.PX - 1) / a.PX;
    // rows enough that every thread has an item, but not so many that the launch leaves CUs without a workgroup
    int TH = std::max(1, std::min(s.Ho, P.slots / P.groups));
    while (TH > 1 && (filters + ((TH - 1) * (int64_t)s.stride + span) * pitch > kFloats || (int64_t)s.N * ((s.Ho + TH - 1) / TH) < 512)) --TH;
    P.TH = TH;
    P.bands = (s.Ho + TH - 1) / TH;
    P.IH = (int)((TH - 1) * (int64_t)s.stride + span);
    P.pitch = (int)pitch;
    const int64_t grid = (int64_t)s.N * P.bands;
    if (grid * P.bands >= (1LL << 32) || grid > 2147483647LL) return a;         // (fast_div's range)
    P.H = s.H; P.W = s.W; P.C_out = s.C_out; P.R = s.R; P.S = s.S; P.stride = s.stride; P.pad = s.pad; P.dil = s.dil;
    P.Ho = s.Ho; P.Wo = s.Wo;
    P.by_pitch = make_fastdiv(P.pitch); P.by_octets = make_fastdiv(P.octets); P.by_groups = make_fastdiv(P.groups);
    P.by_bands = make_fastdiv(P.bands); P.by_K = make_fastdiv(s.R * s.S * s.C_in);
    a.grid = (unsigned)grid;
    a.lds = (size_t)(filters + P.IH * pitch) * 4;
    // Where it is faster, and in launches of 32 workgroups up (with fewer the estimates are worth little).  us, one thread per output
    // against this kernel: 2 x 4 x 1436 x 1 -> 120 under 5x5 at stride 2 7.4 and 51.2, 5 x 8 x 46 x 4 -> 248 under 3x3 at stride 4 6.2 and 15.0,
    // 30 x 17 x 20 x 4 -> 104 under 3x8 at stride 16 15.0 and 22.8; of the drawn layers those that stay took 1.32 x as long
    // here, those that come 0.32 x.
    a.ok = grid >= 32 && few_nhwc_us(P, a.PX, (int64_t)s.R * s.S * s.C_in, grid, a.lds) < 0.9 * one_per_output_nhwc_us(s);
    return a;
}

struct NhwcFPlan {
    NhwcFParams P;
    size_t lds;
    int bands, KS;
    bool ok;
};

NhwcFPlan plan_nhwc_f(const Conv2dShape& s, int esz)
{
    NhwcFPlan a{};
    NhwcFParams& P = a.P;
    const int64_t PB = (int64_t)s.C_in * esz;
    if (PB % 32 != 0 || PB > (1 << 20)) return a;       // whole K steps of 32 bytes per pixel
    const int RS = s.R * s.S;
    P.H = s.H; P.W = s.W; P.C_out = s.C_out; P.R = s.R; P.S = s.S; P.stride = s.stride;
    P.pad = s.pad; P.dil = s.dil; P.Ho = s.Ho; P.Wo = s.Wo;
    P.PB = (int)PB;
    const int64_t IWp = (int64_t)(s.Wo - 1) * s.stride + (int64_t)(s.S - 1) * s.dil + 1;
    if (IWp > 8192) return a;
    P.IWp = (int)IWp;
    // chunk: the largest of 128, 64, 32 bytes per pixel that divides the pixel and whose filters fit the staging
    // slots; then as many output rows per band as the pixel blocks, the slots and LDS allow
    bool found = false;
    for (int cbytes = 128; cbytes >= 32 && !found; cbytes /= 2) {
        if (PB % cbytes != 0) continue;
        P.CB = cbytes;
        P.chunks = (int)(PB / cbytes);
        P.CP = cbytes + 16;
        const int wrow = RS * cbytes;
        P.WPITCH = wrow + 16 + (128 - wrow % 128) % 128;
        P.c16 = cbytes / 16;
        P.wrow16 = wrow / 16;
        if ((int64_t)64 * P.wrow16 >= 65536) continue;  // (exact fast division of the piece index)
        int TH = (kMaxBlocks * 32) / s.Wo;
        if (TH > s.Ho) TH = s.Ho;
        for (; TH >= 1; --TH) {
            const int64_t IH = (int64_t)(TH - 1) * s.stride + (int64_t)(s.R - 1) * s.dil + 1;
            const int64_t xb = IH * P.IWp * P.CP;
            if (IH * P.IWp * P.c16 <= 256 * kXSlots && xb + (int64_t)64 * P.WPITCH <= kLdsBudget) break;
        }
        if (TH < 1) continue;
        const int bands = (s.Ho + TH - 1) / TH;         // equal bands
        TH = (s.Ho + bands - 1) / bands;
        P.TH = TH;
        P.IH = (TH - 1) * s.stride + (s.R - 1) * s.dil + 1;
        found = true;
    }
    if (!found) return a;
    P.x_bytes = (P.IH * P.IWp * P.CP + 15) & ~15;
    a.lds = (size_t)P.x_bytes + (size_t)64 * P.WPITCH;
    a.bands = (s.Ho + P.TH - 1) / P.TH;
    a.KS = P.CB / 32;
    P.by_c16 = make_fastdiv(P.c16);
    P.by_IWp = make_fastdiv(P.IWp);
    P.by_wrow16 = make_fastdiv(P.wrow16);
    P.by_Wo = make_fastdiv(s.Wo);
    a.ok = a.lds <= (size_t)kLdsBudget && s.N <= 65535 && (s.C_out + 63) / 64 <= 65535 &&
           // 32-bit byte offsets inside one image and inside the filters of 64 channels
           (int64_t)s.H * s.W * PB <= 2147483647LL && (int64_t)64 * RS * PB <= 2147483647LL &&
           (int64_t)P.TH * s.Wo <= kMaxBlocks * 32;
    return a;
}

template <int EK, int KS>
hipError_t launch_nhwc_f(const void* x, const void* w, void* y, const NhwcFPlan& a, const Conv2dShape& s, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_nhwc_kernel<EK, KS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBudget);
    if (attr != hipSuccess) return attr;
    dim3 grid((unsigned)a.bands, (unsigned)s.N, (unsigned)((s.C_out + 63) / 64));
    SW_NOTED_LAUNCH(note_kernel("mfma_nhwc_kernel", EK, KS), (mfma_nhwc_kernel<EK, KS>), grid, dim3(256), a.lds, st,
                    static_cast<const unsigned char*>(x), static_cast<const unsigned char*>(w), y, a.P);
    return hipGetLastError();
}

}  // namespace

bool mfma_nhwc_supported(const void* x, const void* w, const Conv2dShape& s, int ek)
{
    return reinterpret_cast<uintptr_t>(x) % 16 == 0 && reinterpret_cast<uintptr_t>(w) % 16 == 0 && plan_nhwc_f(s, elem_size(ek)).ok;
}

hipError_t launch_mfma_nhwc(const void* x, const void* w, void* y, const Conv2dShape& s, int ek, const Epilogue& ep,
                            hipStream_t st)
{
    NhwcFPlan a = plan_nhwc_f(s, elem_size(ek));
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
#define SW_NHWC(EKC)                                                             \
    do {                                                                         \
        if (a.KS == 4) return launch_nhwc_f<EKC, 4>(x, w, y, a, s, st);          \
        if (a.KS == 2) return launch_nhwc_f<EKC, 2>(x, w, y, a, s, st);          \
        return launch_nhwc_f<EKC, 1>(x, w, y, a, s, st);                         \
    } while (0)
    if (ek == kElemF16) SW_NHWC(kElemF16);
    if (ek == kElemBF16) SW_NHWC(kElemBF16);
    SW_NHWC(kElemF32);
#undef SW_NHWC
}

bool few_channels_nhwc_supported(const void* y, const Conv2dShape& s) { return plan_few_nhwc(s, y).ok; }

hipError_t launch_few_channels_nhwc(const void* x, const void* w, void* y, const Conv2dShape& s, int ek, const Epilogue& ep, hipStream_t st)
{
    FewNhwcPlan a = plan_few_nhwc(s, y);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
    // (with the kernel's own 256 bytes a plan may come to more than the 64 KB that a launch has unasked)
#define SW_FEW2(E, C, X)                                                                                                   \
    if (ek == E && s.C_in == C && a.PX == X) {                                                                             \
        static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(few_channels_nhwc_kernel<E, C, X>),  \
                                                           hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);         \
        if (attr != hipSuccess) return attr;                                                                               \
        SW_NOTED_LAUNCH(note_kernel("few_channels_nhwc_kernel", (int)(E), (int)(C), (int)(X)), (few_channels_nhwc_kernel<E, C, X>), dim3(a.grid), dim3(256), \
                        a.lds, st, x, w, y, a.P);                                                                          \
        return hipGetLastError();                                                                                          \
    }
#define SW_FEW(E, C) SW_FEW2(E, C, 1) SW_FEW2(E, C, 4)
    SW_FEW(kElemF32, 1) SW_FEW(kElemF32, 2) SW_FEW(kElemF32, 3) SW_FEW(kElemF32, 4)
    SW_FEW(kElemBF16, 1) SW_FEW(kElemBF16, 2) SW_FEW(kElemBF16, 3) SW_FEW(kElemBF16, 4)
    SW_FEW(kElemF16, 1) SW_FEW(kElemF16, 2) SW_FEW(kElemF16, 3) SW_FEW(kElemF16, 4)
#undef SW_FEW
#undef SW_FEW2
    return hipErrorInvalidValue;
}

hipError_t launch_direct_nhwc(const void* x, const void* w, void* y, const Conv2dShape& s, int ek, const Epilogue& ep,
                              hipStream_t st)
{
    const int64_t total = (int64_t)s.N * s.Ho * s.Wo * s.C_out;
    int64_t blocks = (total + 255) / 256;
    if (blocks > 256 * 64) blocks = 256 * 64;
    if (ek == kElemF16)
        SW_NOTED_LAUNCH(note_kernel("direct_nhwc_kernel", 2), direct_nhwc_kernel<kElemF16>, dim3((unsigned)blocks), dim3(256), 0, st,
                        x, w, y, s, ep);
    else if (ek == kElemBF16)
        SW_NOTED_LAUNCH(note_kernel("direct_nhwc_kernel", 1), direct_nhwc_kernel<kElemBF16>, dim3((unsigned)blocks), dim3(256), 0, st,
                        x, w, y, s, ep);
    else
        SW_NOTED_LAUNCH(note_kernel("direct_nhwc_kernel", 0), direct_nhwc_kernel<kElemF32>, dim3((unsigned)blocks), dim3(256), 0, st,
                        x, w, y, s, ep);
    return hipGetLastError();
}

}  // namespace swconv
