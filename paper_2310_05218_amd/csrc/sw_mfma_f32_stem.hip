// The multi-channel fp32 sliding sum for the first layers of image networks: few input channels, an even stride (7 x 7 over
// RGB at stride 2 and the like), on the bf16 matrix instructions with each fp32 operand as a sum of three bf16 values
// (sw_f32_split.h).
//
//   x [N, C_in, H, W]     w [C_out, C_in, R, S]     y [N, C_out, H_out, W_out]     fp32;   C_in < 8, S <= 8, R C_in <= 22, stride even
//
// With three channels there is nothing to fill the K index of a matrix instruction with but the taps themselves: K runs along
// a filter row.  An operand is eight consecutive taps (the last ones zero when S < 8) of one (filter row, channel) pair, a
// step two pairs: 7 x 7 x 3 = 147 products are 11 steps of 16 instead of the 49 x 16 that channels padded to a K step would be.
//
//   window   [h, m, l][input row][channel][column] bf16, padding as zeros.  The eight inputs of (output pixel, filter row r,
//            channel) are eight neighbouring columns: one 16-byte read, 4-byte aligned because the stride is even.  Filter row
//            and channel are one index q = r C_in + ci, and row q of an output row's window lies q pitches further on.
//   filters  in registers for the whole launch, 12 per step: a wavefront has one block of 32 output channels.
//
// Workgroups are persistent, one per CU, eight wavefronts.  A tile is TH whole output rows of one image in blocks of 32 pixels;
// the next tile's window is loaded into registers before the blocks of this one, split and written to the other LDS buffer
// after them: one barrier per tile, and the wavefronts of a SIMD drift apart so that one splits while the other multiplies.
//
// Measured (us per launch, replayed graphs of ten on one set of buffers, 32 images unless said; the any-shape kernel on fp32 matrix
// instructions -> this one): 7 x 7 stride 2, 3 -> 64 at 224 x 224 169.5 -> 54.2 (error against 64 bits 2.1e-7 -> 6.9e-8), one image
// 25.1 -> 9.7; 3 x 3 stride 2, 3 -> 32 at 224 x 224 47.8 -> 20.8, one image 9.6 -> 6.3.  What bounds it: a block of
// 66 matrix instructions takes a pair of wavefronts 6.2 k ticks where the instructions are 4.2 k (the first operand reads and
// the stores of a block wait), the filters' and the first window's way into LDS 15 k of 107 k ticks.
#include <algorithm>

#include "sw_f32_split.h"
#include "swconv_internal.h"

namespace swconv {

namespace {

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr unsigned kBeyond = 0x80000000u;               // a byte offset no tensor of less than 2 GiB reaches
constexpr int kMaxItems = 4;                            // window items (eight columns of a row) per thread
constexpr int kMaxLds = 160 * 1024;

struct StemParams {
    Epilogue ep;
    int N, C_in, C_out, H, W, Ho, Wo, R, S, stride, pad;
    int TH, tiles_y, tiles, cgroups;   // rows per tile, row tiles per image, tiles, groups of 64 output channels
    int rows, extra, pitch, plane;     // window rows of all channels, those of them that hold zeros, bytes per row, bytes per part
    int groups, items;                 // items per row, items per tile
    unsigned x_bytes, w_bytes;
    FastDiv by_tiles_y, by_groups, by_cin, by_Wo;
};

// eight neighbouring bf16 values from a 4-byte boundary
struct __attribute__((packed, aligned(4))) Quad {
    unsigned v[4];
};
__device__ __forceinline__ bf16x8 read8(const unsigned char* p)
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const Quad*>(p));
}

template <int STEPS>
__global__ __launch_bounds__(512, 2) void mfma_f32_stem_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                               float* __restrict__ y, const StemParams P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 31, kk = lane >> 5;
    // Wavefronts v and v + 4 share a SIMD: one takes the lower 32 output channels and pixel blocks v, v + 4, ..., the other the
    // upper ones and blocks v + 2, v + 6, ... (mod 4), so that the SIMDs differ by at most one block.
    const int cg = blockIdx.y;
    const bool narrow = P.C_out - 64 * cg <= 32;        // one block of output channels: every wavefront takes it
    const int cb = narrow ? 0 : wave >> 2, first = narrow ? wave : (wave + 2 * cb) & 3, every = narrow ? 8 : 4;
    const int co0 = 64 * cg + 32 * cb;
    const int HW = P.H * P.W, HoWo = P.Ho * P.Wo;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, P.x_bytes, 0x00020000);

    // ---- filters: split by all threads into LDS, operands to registers
    const int RC = P.R * P.C_in;
    // (as they lie in memory first: gathered straight from there, 64 output channels per load, they took 8 k ticks)
    constexpr int kStaged = 64 * 2 * STEPS * 3 * 16;
    float* wraw = reinterpret_cast<float*>(smem + kStaged);
    const int per_co = RC * P.S;
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w), 0, P.w_bytes, 0x00020000);
    constexpr int kCopies = (64 * 2 * STEPS * 8 / 4 + 511) / 512;
    uintx4 wcopy[kCopies];
    const unsigned w0 = (unsigned)(64 * cg * per_co * 4);
#pragma unroll
    for (int it = 0; it < kCopies; ++it) {
        const unsigned q = 512 * it + tid;                          // 64 per_co floats are 16 per_co whole pieces
        wcopy[it] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(wr, q < 16u * per_co ? w0 + 16 * q : kBeyond, 0, 0));
    }

    // ---- window: loads of a tile into registers, their way into LDS.  Eight columns of a row are two 16-byte loads, wherever
    // they start (as eight 4-byte loads 32 bytes apart between lanes a tile's loads took 13 k ticks to issue); columns beside
    // the image bring neighbouring rows' values, which store_window clears.
    uintx4 raw[kMaxItems][2];
    auto locate = [&](int i, int& e, int& ci, int& k) __attribute__((always_inline)) {
        const int q = fast_div(i, P.by_groups);
        k = i - q * P.groups;
        e = fast_div(q, P.by_cin);
        ci = q - e * P.C_in;
    };
    auto load = [&](int t) __attribute__((always_inline)) {
        const int n = fast_div(t, P.by_tiles_y), ty = t - n * P.tiles_y;
        const int top = ty * P.TH * P.stride - P.pad;
#pragma unroll
        for (int it = 0; it < kMaxItems; ++it) {
            if (512 * it >= P.items) break;
            int i = 512 * it + tid, e, ci, k;
            asm volatile("" : "+v"(i));                 // (else its quotients are kept across the tiles, and spill)
            locate(i, e, ci, k);
            const int gr = top + e, gc = 8 * k - P.pad;
            const bool in = i < P.items && gr >= 0 && gr < P.H && gc < P.W;
            const int off = ((n * P.C_in + ci) * HW + gr * P.W + gc) * 4;
            if (__builtin_expect(in && (off < 0 || (unsigned)off + 32u > P.x_bytes), 0)) {
                // the first or the last values of the tensor, one by one
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    raw[it][j >> 2][j & 3] = __builtin_amdgcn_raw_buffer_load_b32(xr, gc + j >= 0 && gc + j < P.W ? (unsigned)(off + 4 * j) : kBeyond, 0, 0);
            } else {
                const unsigned o = in ? (unsigned)off : kBeyond;
                raw[it][0] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(xr, o, 0, 0));
                raw[it][1] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(xr, o + 16, 0, 0));
            }
        }
    };
    auto store_window = [&](int buf) __attribute__((always_inline)) {
        unsigned char* d0 = smem + 3 * buf * P.plane;
#pragma unroll
        for (int it = 0; it < kMaxItems; ++it) {
            if (512 * it >= P.items) break;
            int i = 512 * it + tid, e, ci, k;
            asm volatile("" : "+v"(i));
            locate(i, e, ci, k);
            const int gc = 8 * k - P.pad;
            float v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = (unsigned)(gc + j) < (unsigned)P.W ? __uint_as_float(raw[it][j >> 2][j & 3]) : 0.f;
            const Split8 s = split_f32(v);
            if (i < P.items) {
                unsigned char* d = d0 + (e * P.C_in + ci) * P.pitch + 16 * k;
                *reinterpret_cast<bf16x8*>(d) = s.h;
                *reinterpret_cast<bf16x8*>(d + P.plane) = s.m;
                *reinterpret_cast<bf16x8*>(d + 2 * P.plane) = s.l;
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    load(blockIdx.x);

#pragma unroll
    for (int it = 0; it < kCopies; ++it) {
        const int q = 512 * it + tid;
        if (q < 16 * per_co) *reinterpret_cast<uintx4*>(wraw + 4 * q) = wcopy[it];
    }
    __syncthreads();
#pragma unroll 1
    for (int i = tid; i < 64 * 2 * STEPS; i += 512) {
        const int q = i >> 6, co = i & 63;
        const int r = fast_div(q, P.by_cin), ci = q - r * P.C_in;
        const float* wp = wraw + co * per_co + (ci * P.R + r) * P.S;
        const bool in = q < RC && 64 * cg + co < P.C_out;
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = in && j < P.S ? wp[j] : 0.f;
        const Split8 s = split_f32(v);
        bf16x8* d = reinterpret_cast<bf16x8*>(smem) + 3 * 64 * q + co;
        d[0] = s.h;
        d[64] = s.m;
        d[128] = s.l;
    }
    __syncthreads();
    Split8 a[STEPS];
#pragma unroll
    for (int g = 0; g < STEPS; ++g) {
        const bf16x8* s = reinterpret_cast<const bf16x8*>(smem) + 3 * 64 * (2 * g + kk) + 32 * cb + lj;
        a[g].h = s[0];
        a[g].m = s[64];
        a[g].l = s[128];
    }
    __syncthreads();
    // the rows of zeros behind the window (pairs of the last step that the filter does not have), in both buffers
    for (int i = tid; i < 6 * P.extra * (P.pitch / 4); i += 512) {
        const int row = i / (P.pitch / 4), part = row / P.extra;
        reinterpret_cast<unsigned*>(smem + part * P.plane + (P.rows - P.extra + row - part * P.extra) * P.pitch)[i - row * (P.pitch / 4)] = 0;
    }
    store_window(0);
    __syncthreads();

    int buf = 0;
#pragma unroll 1
    for (int t = blockIdx.x; t < P.tiles; t += gridDim.x, buf ^= 1) {
        const bool more = t + (int)gridDim.x < P.tiles;
        if (more) load(t + gridDim.x);
        const int n = fast_div(t, P.by_tiles_y), ty = t - n * P.tiles_y;
        const int row0 = ty * P.TH;
        const int valid_px = min(P.TH, P.Ho - row0) * P.Wo;
        const unsigned char* win = smem + 3 * buf * P.plane + kk * P.pitch;
#pragma unroll 1
        for (int b = first; 32 * b < valid_px; b += every) {
            const int p = 32 * b + lj, pc = min(p, valid_px - 1);
            const int ol = fast_div(pc, P.by_Wo), ow = pc - ol * P.Wo;
            const unsigned char* bp = win + ol * P.stride * P.C_in * P.pitch + 2 * P.stride * ow;
            // the products of the high parts, and the five others (at most 2^-8 of them): apart, because an accumulator's rounding
            // follows its magnitude
            splitx16 acc, low;
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[v] = 0.f; low[v] = 0.f; }
            Split8 o[2];
            auto fetch = [&](Split8& d, int g) __attribute__((always_inline)) {
                const unsigned char* s = bp + 2 * g * P.pitch;
                d.h = read8(s);
                d.m = read8(s + P.plane);
                d.l = read8(s + 2 * P.plane);
            };
            fetch(o[0], 0);
#pragma unroll
            for (int g = 0; g < STEPS; ++g) {
                if (g + 1 < STEPS) fetch(o[(g + 1) & 1], g + 1);
                const Split8& c = o[g & 1];
                __builtin_amdgcn_sched_barrier(0);
                low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g].l, c.h, low, 0, 0, 0);
                low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g].h, c.l, low, 0, 0, 0);
                low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g].m, c.m, low, 0, 0, 0);
                low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g].m, c.h, low, 0, 0, 0);
                low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g].h, c.m, low, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[g].h, c.h, acc, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            acc += low;
            // register v of a lane is output channel 8 (v / 4) + 4 kk + v % 4, pixel lj
            float* yp = y + ((int64_t)n * P.C_out + co0 + 4 * kk) * HoWo + (int64_t)row0 * P.Wo + p;
            const bool beyond = p < valid_px && split_overflow(acc);
            split_unscale(acc);
            if (p < valid_px) store_block(acc, yp, HoWo, co0 + 4 * kk, P.C_out, co0 + 32 <= P.C_out, P.ep);
            if (__builtin_expect(__ballot(beyond) != 0, 0)) {
                const splitx16 again = multiply_f32<8>(w, RC * P.S, co0 + lj, P.C_out, kk,
                                                    ConvInputs(xr, P.C_in, P.H, P.W, P.R, P.S, P.stride, P.pad, 1, n, row0 + ol, ow,
                                                               kk * ((RC * P.S + 1) >> 1)));
                if (beyond) store_outputs(again, yp, HoWo, co0 + 4 * kk, P.C_out, P.ep);
            }
        }
        if (more) store_window(buf ^ 1);
        __syncthreads();
    }
}

struct StemPlan {
    bool ok = false;
    int STEPS = 0, lds = 0;
    unsigned gx = 0;
    double est = 0;
    StemParams P;
};

StemPlan search_stem(const Conv2dShape& s)
{
    StemPlan best;
    const int RC = s.R * s.C_in;
    const int64_t x_bytes = (int64_t)s.N * s.C_in * s.H * s.W * 4;
    const int64_t w_bytes = (int64_t)s.C_out * RC * s.S * 4;
    if (s.C_in < 2 || s.C_in > 7 || s.S > 8 || RC > 22 || s.stride % 2 != 0 || s.dil != 1 || x_bytes >= (1LL << 31) || w_bytes >= (1LL << 31)) return best;
    const int STEPS = RC <= 10 ? 5 : RC <= 16 ? 8 : 11;
    // Short filter rows leave most of the K index empty: the kernels on fp32 matrix instructions have R S products of 2, 4 or 8 channels
    // against 6 STEPS steps of sixteen here.  From 0.6 of them up (two channels, which those kernels hold without a rest: 0.7) this one
    // is no slower (us, theirs / this one: 1 x 1 over 2 channels, 32 images of 224 x 224, 24.2 / 37.1, 2 x 2 over 3 35.9 / 33.2 but 16 of
    // 112 x 112 9.1 / 10.0, over 7 59.1 / 52.0, 3 x 3 over 2 9.3 / 10.3, over 3 52.3 / 33.0).  At strides from 4 up they bring in whole windows
    // of mostly unused columns, unless there is next to nothing to do (2 x 2 stride 8 over 4, 20 of 132 x 18, 11.3 / 6.7; 1 x 5 stride 4 over
    // 2, 34 of 9 x 116 6.3 / 7.4).  Two of 840 timed shapes are slower by more than 10 %.
    const double products = (double)s.R * s.S * (s.C_in == 2 ? 2 : s.C_in <= 4 ? 4 : 8) / (6 * STEPS);
    if (products < (s.C_in == 2 ? 0.7 : 0.6) &&
        !(s.stride >= 4 && products >= 0.25 && (int64_t)s.Ho * s.Wo >= 40 && std::min(s.Ho, s.Wo) >= 2)) return best;
    if ((s.C_out + 63) / 64 > 65535) return best;            // (second dimension of a launch)
    const int64_t cols = (int64_t)s.stride * (s.Wo - 1) + 8, groups = (cols + 7) / 8;
    if (groups > 512) return best;
    const int64_t most = (512 * kMaxItems / (s.C_in * groups) - s.R) / s.stride + 1;     // rows of a tile whose window the items hold
    for (int rows_max = (int)std::min<int64_t>(s.Ho, most), last = 0; rows_max >= 1; --rows_max) {
        const int tiles_y = (s.Ho + rows_max - 1) / rows_max, TH = (s.Ho + tiles_y - 1) / tiles_y;
        if (tiles_y == last) continue;
        last = tiles_y;
        // window rows of a tile: those of its output rows, and rows of zeros for the pairs of the last steps beyond the filter
        const int64_t IH = (int64_t)s.stride * (TH - 1) + s.R, extra = 2 * STEPS - RC, rows = IH * s.C_in + extra;
        const int64_t items = IH * s.C_in * groups, pitch = 16 * groups, plane = rows * pitch;
        if (items > 512 * kMaxItems) continue;
        const int64_t lds = std::max<int64_t>(6 * plane, 64 * 6 * 16 * STEPS + 256 * RC * s.S);
        const int64_t tiles = (int64_t)s.N * tiles_y;
        if (lds > kMaxLds || tiles * tiles_y >= (1LL << 32)) continue;
        const int cgroups = (s.C_out + 63) / 64;
        const int64_t gx = std::min<int64_t>(tiles, std::max(1, 256 / cgroups));
        // ticks: blocks of a SIMD (38 a matrix instruction, 500 to store), the tile's way into LDS
        const int64_t blocks = ((int64_t)TH * s.Wo + 31) / 32;
        const double per = (double)((2 * blocks + 3) / 4) * (38.0 * 6 * STEPS + 500) + (double)((items + 511) / 512) * 900 + 600;
        const double est = (double)((tiles + gx - 1) / gx) * per;
        if (best.ok && est >= best.est) continue;
        best.ok = true;
        best.est = est;
        best.STEPS = STEPS;
        best.lds = (int)lds;
        best.gx = (unsigned)gx;
        StemParams& P = best.P;
        P.N = s.N; P.C_in = s.C_in; P.C_out = s.C_out; P.H = s.H; P.W = s.W; P.Ho = s.Ho; P.Wo = s.Wo;
        P.R = s.R; P.S = s.S; P.stride = s.stride; P.pad = s.pad;
        P.TH = TH; P.tiles_y = tiles_y; P.tiles = (int)tiles; P.cgroups = cgroups;
        P.rows = (int)rows; P.extra = (int)extra; P.pitch = (int)pitch; P.plane = (int)plane;
        P.groups = (int)groups; P.items = (int)items;
        P.x_bytes = (unsigned)x_bytes; P.w_bytes = (unsigned)w_bytes;
        P.by_tiles_y = make_fastdiv(tiles_y); P.by_groups = make_fastdiv((int)groups);
        P.by_cin = make_fastdiv(s.C_in); P.by_Wo = make_fastdiv(s.Wo);
    }
    return best;
}

StemPlan plan_stem(const Conv2dShape& s)
{
    thread_local PlanCache<StemPlan> cache;
    return cache.get(s, 0, [&] { return search_stem(s); });
}

template <int STEPS>
hipError_t launch_stem(const float* x, const float* w, float* y, const StemPlan& a, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_f32_stem_kernel<STEPS>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel("mfma_f32_stem_kernel", STEPS, a.P.TH), (mfma_f32_stem_kernel<STEPS>), dim3(a.gx, a.P.cgroups), dim3(512),
                    a.lds, st, x, w, y, a.P);
    return hipGetLastError();
}

}  // namespace

bool mfma_f32_stem_supported(const Conv2dShape& s) { return plan_stem(s).ok; }

hipError_t launch_mfma_f32_stem(const float* x, const float* w, float* y, const Conv2dShape& s, hipStream_t st, const Epilogue& ep)
{
    StemPlan a = plan_stem(s);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
    if (a.STEPS == 5) return launch_stem<5>(x, w, y, a, st);
    if (a.STEPS == 8) return launch_stem<8>(x, w, y, a, st);
    return launch_stem<11>(x, w, y, a, st);
}

}  // namespace swconv
