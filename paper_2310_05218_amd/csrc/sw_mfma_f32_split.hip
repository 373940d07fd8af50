// The multi-channel fp32 sliding sum with nine taps (3 x 3, any stride, padding and dilation) on the bf16 matrix
// instructions, each fp32 operand as a sum of three bf16 values (sw_f32_split.h): six v_mfma_f32_32x32x16_bf16 per tap and
// 16 channels take 192 cycles where eight v_mfma_f32_32x32x2_f32 take 512.
//
//   x [N, C_in, H, W]     w [C_out, C_in, 3, 3]     y [N, C_out, H_out, W_out]     fp32
//
// A workgroup owns tiles of 32 output channels x up to 256 PB output pixels (whole rows of one image, or several whole small
// images) and walks over them; the reduction runs in chunks of 16 channels x nine taps.  Splitting a value costs about seven
// vector instructions, so it is done once per workgroup, on the way into LDS, by wavefronts that do nothing else, under the
// matrix instructions of the others:
//
//   filters  [tap][h, m, l][channel octet][output channel] of 16 bytes: eight channels of one tap.  The eight channels of an
//            octet x nine taps of an output channel are 288 consecutive bytes of w: a lane loads them with 18 16-byte loads
//            a chunk period ahead and gathers the taps from its registers.
//   window   [h, m, l][channel octet][cell] of 16 bytes: the rectangle of input pixels the tile touches, padding as zeros.
//            A lane loads eight channels of one cell (consecutive lanes: consecutive pixels).
//
// Both layouts give the matrix operands as conflict-free 16-byte reads; tap shift, stride and dilation are in the address.
// The first eight (PH = 4: three) wavefronts multiply, the next PH split filters, the last 4 - PH (PH = 4: one) split windows.  There are two window stages and PH + 1
// filter stages: a filter wavefront has PH chunk periods for its chunk (PH chunks are under way at a time), which is what
// keeps small tiles, whose periods are short, supplied; large windows leave room for PH = 1 only.  One barrier per chunk.
//
// Measured (us per launch, replayed graphs of ten on one set of buffers, batch 32 unless said, the fp32-instruction kernels -> this
// one): 64 -> 64 at 56 x 56 75.4 -> 49.7, 128 -> 128 at 28 x 28 87.1 -> 45.0, 256 -> 256 at 14 x 14 84.4 -> 45.3, 512 -> 512 at 7 x 7
// 103.5 -> 54.8, one image of 64 -> 64 at 56 x 56 21.1 -> 10.2, five of 96 -> 136 at 35 x 35 39.0 -> 17.8.  (Smaller launches are the few-tiles kernel's
// now: one image of 256 -> 256 at 14 x 14 39.4 -> 17.4 here and 10.6 there, of 512 -> 512 at 7 x 7 73.9 -> 29.8 and 16.1.)
// What bounds it: 256 pixels x PB of a tile are never quite full (13 of 16 blocks in the first case), the first chunk's way
// through LDS (7 us) and the stores of a tile that nothing overlaps, and a clock of 1.8-1.9 GHz under the bf16 instructions.  With
// parts left out, the first case takes 14 us for launch, barriers and window loads, 34 with the matrix instructions of three blocks
// per SIMD besides (30 cycles each: their chains cost nothing), 36 with their operand reads, 44 with the stores and the thirteenth
// block, 50 with the splitting.  (The thirteenth block in quarters over four SIMDs, on 16 x 16 x 32 instructions, gained nothing over
// leaving out the dead ones: each quarter reads as much of LDS as the block.)  Single images: about 2 k ticks a
// chunk, most of it the filter loads (64 lanes 288 bytes apart are 64 lines a load, 1.2 k ticks a chunk).  Three wavefronts share
// the taps of single blocks: with a tile's only block on one wavefront 512 -> 512 at 7 x 7 took 40.2 us where it took 29.8, 3 x 344 -> 88
// at 9 x 9 28.2 where it took 20.1.
#include <algorithm>

#include "sw_f32_split.h"
#include "swconv_internal.h"

namespace swconv {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr unsigned kBeyond = 0x80000000u;               // a byte offset no tensor of less than 2 GiB reaches
constexpr int kTaps = 9;
constexpr int kFilterStage = kTaps * 3 * 2 * 32 * 16;   // 27 KB

// Multiplying wavefronts: two per SIMD, so that one reads operands while the other multiplies.  With PH = 4, for launches of at
// most one tile of one block per workgroup, three share the block, a third of the taps each, and the filter wavefronts have
// registers for a second chunk in flight (eight wavefronts instead of twelve).
constexpr int mul_waves(int PH) { return PH == 4 ? 3 : 8; }
constexpr int win_waves(int PH) { return PH == 4 ? 1 : 4 - PH; }

// cells of a window that fit beside PH + 1 filter stages
constexpr int max_cells(int PH) { return PH == 1 ? 528 : PH == 2 ? 400 : 112; }
// cells of a window lane's items: its byte offsets wait in LDS for the rolled loop that computes them
constexpr int lane_items(int PH) { return (2 * max_cells(PH) + 64 * win_waves(PH) - 1) / (64 * win_waves(PH)); }
constexpr int lds_bytes(int PH) { return (PH + 1) * kFilterStage + 2 * 96 * max_cells(PH) + 256 * win_waves(PH) * lane_items(PH); }

struct SplitParams {
    Epilogue ep;
    int N, C_in, C_out, H, W, Ho, Wo, R, S, stride, pad, dil;
    int NI, TH, tiles_y;           // images and output rows per tile, row tiles per image
    int IW, cells_img, WC;         // window columns, cells of one image, cells of a tile
    int px_tiles, tiles;           // pixel tiles; pixel tiles x blocks of 32 output channels
    int chunks;
    unsigned x_bytes, w_bytes;
    int tap_off[kTaps];            // byte offset of a tap's cell from the pixel's first cell
    FastDiv by_px_tiles, by_tiles_y, by_cells_img, by_IW, by_thwo, by_Wo;
};

// barrier without the fence of __syncthreads (which would wait for the global stores and loads in flight)
__device__ __forceinline__ void chunk_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int PH, int PB>
__global__ __launch_bounds__(64 * (mul_waves(PH) + PH + win_waves(PH)), mul_waves(PH) == 8 ? 3 : 2) void mfma_f32_split_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                                float* __restrict__ y, const SplitParams P)
{
    constexpr int CW = mul_waves(PH);
    constexpr bool kShared = PH == 4;                   // one block per tile: the multiplying wavefronts share it, a row of taps each
    constexpr int CELLS = max_cells(PH);
    constexpr int OCT = CELLS * 16, PLANE = 2 * OCT, WSTAGE = 3 * PLANE;
    constexpr int WIN0 = (PH + 1) * kFilterStage;
    constexpr int TABLE0 = WIN0 + 2 * WSTAGE;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int my_tiles = (P.tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
    const int T = my_tiles * P.chunks;                  // chunks of all of this workgroup's tiles, one barrier each
    const int HW = P.H * P.W;

    // the splitting wavefronts first: a matrix instruction needs an issue slot every 32 cycles only
    if (wave >= CW) __builtin_amdgcn_s_setprio(3);
    if (wave >= CW + PH) {
        // ------------------------------------------------------------------------------------------ windows
        constexpr int NW = win_waves(PH), IT = lane_items(PH);
        const int q0 = (wave - CW - PH) * 64 + lane;
        unsigned* table = reinterpret_cast<unsigned*>(smem + TABLE0) + (wave - CW - PH) * 64 * IT + lane;
        const int items = 2 * P.WC;
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, P.x_bytes, 0x00020000);
        unsigned base[IT];
        float raw0[IT][8], raw1[IT][8];                 // two chunks in flight
        auto locate = [&](int t) __attribute__((always_inline)) {
            const int pt = t - fast_div(t, P.by_px_tiles) * P.px_tiles;
            const int ig = fast_div(pt, P.by_tiles_y), ty = pt - ig * P.tiles_y;
            const int n0 = ig * P.NI, top = ty * P.TH * P.stride - P.pad;
            // (a rolled loop, its results through LDS: unrolled, the code itself took longer to fetch than to run)
#pragma unroll 1
            for (int it = 0; it < IT; ++it) {
                const int q = q0 + 64 * NW * it;
                const int oct = q >= P.WC, cell = q - (oct ? P.WC : 0);
                const int i = fast_div(cell, P.by_cells_img), rem = cell - i * P.cells_img;
                const int e = fast_div(rem, P.by_IW), f = rem - e * P.IW;
                const int gr = top + e, gc = f - P.pad, n = n0 + i;
                const bool in = q < items && n < P.N && gr >= 0 && gr < P.H && gc >= 0 && gc < P.W;
                table[64 * it] = in ? (unsigned)(((n * P.C_in + 8 * oct) * HW + gr * P.W + gc) * 4) : kBeyond;
            }
#pragma unroll
            for (int it = 0; it < IT; ++it) base[it] = table[64 * it];
        };
        int c = 0, t = blockIdx.x;                      // the next chunk to load
        auto load = [&](float (&raw)[IT][8]) __attribute__((always_inline)) {
            const int ci0 = 16 * c;
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                if (64 * NW * it >= items) break;
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    raw[it][j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xr, base[it] + (unsigned)((ci0 + j) * HW * 4), 0, 0));
            }
        };
        // loads the next chunk, if there is one, and steps on
        int issued = 0;
        auto load_next = [&](float (&raw)[IT][8]) __attribute__((always_inline)) {
            if (issued >= T) return;
            if (c == 0) locate(t);
            load(raw);
            ++issued;
            if (++c == P.chunks) { c = 0; t += gridDim.x; }
        };
        int cc = 0;                                     // the next chunk to convert
        auto convert = [&](int i, float (&raw)[IT][8]) __attribute__((always_inline)) {
            unsigned char* sw = smem + WIN0 + (i & 1) * WSTAGE;
            const int beyond = P.C_in - 16 * cc;
            if (++cc == P.chunks) cc = 0;
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                if (64 * NW * it >= items) break;
                const int q = q0 + 64 * NW * it;
                if (beyond < 16) {
#pragma unroll
                    for (int j = 0; j < 8; ++j)
                        if (j >= beyond - (q >= P.WC ? 8 : 0)) raw[it][j] = 0.f;
                }
                const Split8 s = split_f32(raw[it]);
                if (q < items) {
                    unsigned char* d = sw + (q >= P.WC ? OCT + (q - P.WC) * 16 : q * 16);
                    *reinterpret_cast<bf16x8*>(d) = s.h;
                    *reinterpret_cast<bf16x8*>(d + PLANE) = s.m;
                    *reinterpret_cast<bf16x8*>(d + 2 * PLANE) = s.l;
                }
            }
        };
        load_next(raw0);
        load_next(raw1);
#pragma unroll 1
        for (int i = 0; i < T; i += 2) {
            convert(i, raw0);
            chunk_barrier();
            load_next(raw0);
            if (i + 1 < T) {
                convert(i + 1, raw1);
                chunk_barrier();
                load_next(raw1);
            }
        }
        if constexpr (kShared) {                        // (the barriers around the partial sums)
            chunk_barrier();
            chunk_barrier();
        }
        return;
    }

    if (wave >= CW) {
        // ------------------------------------------------------------------------------------------ filters
        const int f = wave - CW;
        const int co = lane & 31, oct = lane >> 5;
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w), 0, P.w_bytes, 0x00020000);
        constexpr bool kAhead = PH == 4;
        floatx4 raw0[18], raw1[kAhead ? 18 : 1];
        // pieces first .. last - 1 of the 18 of this lane's run of chunk i
        auto load = [&](int i, auto& raw, int first, int last) __attribute__((always_inline)) {
            const int k = i / P.chunks, c = i - k * P.chunks;
            const int t = blockIdx.x + k * gridDim.x;
            const int cog = 32 * fast_div(t, P.by_px_tiles) + co, ci = 16 * c + 8 * oct;
            const unsigned off = i < T && cog < P.C_out && ci < P.C_in ? (unsigned)((cog * P.C_in + ci) * (kTaps * 4)) : kBeyond;
#pragma unroll
            for (int k4 = first; k4 < last; ++k4)
                raw[k4] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off + 16 * k4, 0, 0));
        };
        auto chunk = [&](int i, floatx4 (&raw)[18], auto& next) __attribute__((always_inline)) {
            unsigned char* sf = smem + (i % (PH + 1)) * kFilterStage + oct * 512 + co * 16;
            const int c = i - (i / P.chunks) * P.chunks;
            const int lim = P.C_in - 16 * c - 8 * oct;
#pragma unroll
            for (int ph = 0; ph < PH; ++ph) {
                if (i - PH + ph >= 0) chunk_barrier();
                if (ph == 0) {
                    if (16 * c + 16 > P.C_in) {                     // the run of the last channels reaches into the next filter
#pragma unroll
                        for (int q = 0; q < 72; ++q)
                            if (q / kTaps >= lim) raw[q / 4][q % 4] = 0.f;
                    }
                }
#pragma unroll
                for (int tap = kTaps * ph / PH; tap < kTaps * (ph + 1) / PH; ++tap) {
                    float v[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) v[j] = raw[(kTaps * j + tap) / 4][(kTaps * j + tap) % 4];
                    const Split8 s = split_f32(v);
                    *reinterpret_cast<bf16x8*>(sf + tap * 3072) = s.h;
                    *reinterpret_cast<bf16x8*>(sf + tap * 3072 + 1024) = s.m;
                    *reinterpret_cast<bf16x8*>(sf + tap * 3072 + 2048) = s.l;
                }
                    // the next chunk's loads: 64 lanes 288 bytes apart take 64 ticks a load to issue; in one piece they made every
                // third period of a small tile twice as long
                if constexpr (kAhead) load(i + PH, next, 18 * ph / PH, 18 * (ph + 1) / PH);
            }
            if constexpr (!kAhead) load(i + PH, raw, 0, 18);
        };
        load(f, raw0, 0, 18);
        if constexpr (kAhead) {
#pragma unroll 1
            for (int i = f; i < T; i += 2 * PH) {
                chunk(i, raw0, raw1);
                if (i + PH < T) chunk(i + PH, raw1, raw0);
            }
        } else {
#pragma unroll 1
            for (int i = f; i < T; i += PH) chunk(i, raw0, raw1);
        }
        // (chunk i of this wavefront passed the barriers up to i - 1)
        const int last = f < T ? f + ((T - 1 - f) / PH) * PH : 0;
#pragma unroll 1
        for (int b = last; b < T; ++b) chunk_barrier();
        if constexpr (kShared) {
            chunk_barrier();
            chunk_barrier();
        }
        return;
    }

    // ---------------------------------------------------------------------------------------------- products
    const int lj = lane & 31, kk = lane >> 5;
    const int HoWo = P.Ho * P.Wo, thwo = P.TH * P.Wo;
    int i = 0;
#pragma unroll 1
    for (int t = blockIdx.x; t < P.tiles; t += gridDim.x) {
        const int cb = fast_div(t, P.by_px_tiles), pt = t - cb * P.px_tiles;
        const int ig = fast_div(pt, P.by_tiles_y), ty = pt - ig * P.tiles_y;
        const int n0 = ig * P.NI, row0 = ty * P.TH, co0 = 32 * cb;
        const int valid_px = P.NI > 1 ? min(P.NI, P.N - n0) * HoWo : min(P.TH, P.Ho - row0) * P.Wo;
        int pix[PB];                                    // (a lane without a pixel multiplies cell 0)
        int nlive = 0;
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            const int first = kShared ? 0 : 32 * (CW * b + wave), p = first + lj;
            if (first < valid_px) nlive = b + 1;
            const int im = fast_div(p, P.by_thwo), rem = p - im * thwo;
            const int ol = fast_div(rem, P.by_Wo), ow = rem - ol * P.Wo;
            pix[b] = (p < valid_px ? 16 * (im * P.cells_img + (ol * P.IW + ow) * P.stride) : 0) + kk * OCT;
        }
        // the products of the high parts, and the five others (at most 2^-8 of them): apart, because an accumulator's
        // rounding follows its magnitude -- a third of the error of one accumulator for all six
        splitx16 acc[PB], low[PB];
#pragma unroll
        for (int b = 0; b < PB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[b][v] = 0.f; low[b][v] = 0.f; }

#pragma unroll 1
        for (int c = 0; c < P.chunks; ++c, ++i) {
            chunk_barrier();
            if (nlive == 0) continue;
            const unsigned char* sf = smem + (i % (PH + 1)) * kFilterStage + kk * 512 + lj * 16;
            const unsigned char* sw = smem + WIN0 + (i & 1) * WSTAGE;
            auto split_at = [](const unsigned char* p, int plane) __attribute__((always_inline)) {
                return Split8{*reinterpret_cast<const bf16x8*>(p), *reinterpret_cast<const bf16x8*>(p + plane), *reinterpret_cast<const bf16x8*>(p + 2 * plane)};
            };
            auto filters = [&](int tap) __attribute__((always_inline)) { return split_at(sf + tap * 3072, 1024); };
            auto pixels = [&](int tap, int b) __attribute__((always_inline)) { return split_at(sw + (pix[b] + P.tap_off[tap]), PLANE); };
            struct Ops {
                Split8 a, b;
            };
            auto fetch = [&](Ops& o, int tap) __attribute__((always_inline)) {
                o.a = filters(tap);
                o.b = pixels(tap, 0);
            };
            auto mul = [&](const Split8& f, const Split8& v, int b) __attribute__((always_inline)) {
                // in ascending order of magnitude
                low[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.l, v.h, low[b], 0, 0, 0);
                low[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.h, v.l, low[b], 0, 0, 0);
                low[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.m, v.m, low[b], 0, 0, 0);
                low[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.m, v.h, low[b], 0, 0, 0);
                low[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.h, v.m, low[b], 0, 0, 0);
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.h, v.h, acc[b], 0, 0, 0);
            };
            if constexpr (kShared) {
                Ops o[3];
#pragma unroll
                for (int j = 0; j < 3; ++j) fetch(o[j], 3 * wave + j);
#pragma unroll
                for (int j = 0; j < 3; ++j) mul(o[j].a, o[j].b, 0);
            } else if constexpr (PB == 2) {
                // (registers for one set of operands: the other wavefront of the SIMD covers the reads.)  A wavefront whose second
                // block lies beyond the tile -- three of eight where a tile has 13 blocks of 16 -- leaves its products out: they took the
                // SIMD's other wavefront a sixth of its matrix time (64 -> 64 at 56 x 56, batch 12 of 48 -> 64, 22 of 88 -> 24 at
                // 47 x 54 with dilation 2: 51.6 -> 49.7, 20.9 -> 17.6, 32.4 -> 26.3 us).  The test is on the tile's size only, the same for
                // all lanes; a lone block in a copy of the loop took 54 registers more than there are.
                const bool two = nlive == 2;
#pragma unroll
                for (int tap = 0; tap < kTaps; ++tap) {
                    const Split8 f = filters(tap);
                    mul(f, pixels(tap, 0), 0);
                    if (two) mul(f, pixels(tap, 1), 1);
                }
            } else {
                Ops o[2];
                fetch(o[0], 0);
#pragma unroll
                for (int tap = 0; tap < kTaps; ++tap) {
                    if (tap + 1 < kTaps) fetch(o[(tap + 1) & 1], tap + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    mul(o[tap & 1].a, o[tap & 1].b, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
#pragma unroll
        for (int b = 0; b < PB; ++b) acc[b] += low[b];
        if constexpr (kShared) {
            // the parts meet in LDS, over stages that everybody has left (one tile per workgroup)
            chunk_barrier();
            float* part = reinterpret_cast<float*>(smem);
            if (wave > 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) part[((wave - 1) * 16 + v) * 64 + lane] = acc[0][v];
            }
            chunk_barrier();
            if (wave > 0) return;
#pragma unroll
            for (int q = 0; q < CW - 1; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][v] += part[(q * 16 + v) * 64 + lane];
        }

        // ---- store: register v of a lane is output channel 8 (v / 4) + 4 kk + v % 4, pixel lj
#pragma unroll
        for (int b = 0; b < PB; ++b) {
            const int p = (kShared ? 0 : 32 * (CW * b + wave)) + lj;
            const int im = fast_div(p, P.by_thwo), rem = p - im * thwo;
            const int ol = fast_div(rem, P.by_Wo), ow = rem - ol * P.Wo;
            float* yp = y + ((int64_t)(n0 + im) * P.C_out + co0 + 4 * kk) * HoWo + (row0 + ol) * P.Wo + ow;
            const bool beyond = p < valid_px && split_overflow(acc[b]);
            split_unscale(acc[b]);
            if (p < valid_px) store_block(acc[b], yp, HoWo, co0 + 4 * kk, P.C_out, co0 + 32 <= P.C_out, P.ep);
            if (__builtin_expect(__ballot(beyond) != 0, 0)) {
                const int per = P.C_in * kTaps;
                const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, P.x_bytes, 0x00020000);
                const splitx16 again = multiply_f32<8>(w, per, co0 + lj, P.C_out, kk,
                                                    ConvInputs(xr, P.C_in, P.H, P.W, P.R, P.S, P.stride, P.pad, P.dil, n0 + im, row0 + ol, ow,
                                                               kk * ((per + 1) >> 1)));
                if (beyond) store_outputs(again, yp, HoWo, co0 + 4 * kk, P.C_out, P.ep);
            }
        }
    }
}

struct SplitPlan {
    bool ok = false;
    int PH = 0, PB = 0;
    unsigned grid = 0;
    double est = 0;
    SplitParams P;
};

SplitPlan search_split(const Conv2dShape& s)
{
    SplitPlan best;
    if (s.R * s.S != kTaps) return best;
    const int64_t x_bytes = (int64_t)s.N * s.C_in * s.H * s.W * 4, w_bytes = (int64_t)s.C_out * s.C_in * kTaps * 4;
    // (the last chunk's channels that do not exist are read and cleared: their offsets stay below 2^31 as well)
    if (x_bytes + 60LL * s.H * s.W >= (1LL << 31) || w_bytes >= (1LL << 31)) return best;
    const int64_t IW = (int64_t)(s.Wo - 1) * s.stride + (int64_t)(s.S - 1) * s.dil + 1;
    if (IW > 528) return best;
    const int chunks = (s.C_in + 15) / 16, co_blocks = (s.C_out + 31) / 32;
    auto consider = [&](int NI, int tiles_y) {
        const int TH = (s.Ho + tiles_y - 1) / tiles_y;
        if ((s.Ho + TH - 1) / TH != tiles_y) return;
        const int64_t px = (int64_t)NI * TH * s.Wo;
        const int64_t IH = (int64_t)(TH - 1) * s.stride + (int64_t)(s.R - 1) * s.dil + 1;
        const int64_t WC = NI * IH * IW;
        const int64_t blocks = (px + 31) / 32;
        if (blocks > 16) return;
        const int64_t px_tiles = (int64_t)((s.N + NI - 1) / NI) * tiles_y, tiles = px_tiles * co_blocks;
        if (tiles * px_tiles >= (1LL << 32)) return;        // (fast_div's range)
        // A stride-2 window holds four cells per output pixel, and splitting those takes longer than multiplying: with one
        // tile per workgroup still the faster kernel (128 -> 128 at 56 x 56, 8 images: 22.2 us against 37.0), beyond that
        // not (64 -> 128, 32 images: 58 against 51 when last tried).
        if (s.stride > 1 && tiles > 256) return;
        for (int PH : {1, 2, 4}) {
            // PH = 4 adds up one block of one tile per workgroup.  Measured on single images against PH = 3 and a block per
            // wavefront, when it took its place: 256 -> 256 at 14 x 14 23.6 -> 23.1, 512 -> 512 at 7 x 7 40.2 -> 31.3, 16 x 128 -> 32 at
            // 17 x 17 14.6 -> 12.7.
            if (PH == 4 && (blocks > 1 || tiles > 256)) continue;
            const int64_t PB = (blocks + mul_waves(PH) - 1) / mul_waves(PH);
            if (WC > max_cells(PH) || PB > (PH == 1 ? 2 : 1)) continue;
            // ticks of a chunk: the matrix instructions of a SIMD (40 each with their operand reads), a filter wavefront's
            // share, a window wavefront's items of 64 cells -- as time stamps showed them
            const int NW = win_waves(PH), per_simd = (int)((blocks + 3) / 4);
            const double mul = 40.0 * 6 * (PH == 4 ? 3 : kTaps) * per_simd + 300;
            const double fil = PH == 4 ? 1500.0 : 6100.0 / PH, win = (double)((2 * WC + 64 * NW - 1) / (64 * NW)) * (PH == 4 ? 600 : 950) + (PH == 4 ? 400 : 600);
            const double per = std::max(mul, std::max(fil, win)) * chunks;
            const double est = (double)((tiles + 255) / 256) * (per + 1500.0 * per_simd) + 12000;
            if (best.ok && est >= best.est) continue;
            best.ok = true;
            best.est = est;
            best.PH = PH; best.PB = (int)PB;
            best.grid = (unsigned)std::min<int64_t>(tiles, 256);
            SplitParams& P = best.P;
            P.N = s.N; P.C_in = s.C_in; P.C_out = s.C_out; P.H = s.H; P.W = s.W; P.Ho = s.Ho; P.Wo = s.Wo;
            P.R = s.R; P.S = s.S; P.stride = s.stride; P.pad = s.pad; P.dil = s.dil;
            P.NI = NI; P.TH = TH; P.tiles_y = tiles_y;
            P.IW = (int)IW; P.cells_img = (int)(IH * IW); P.WC = (int)WC;
            P.px_tiles = (int)px_tiles; P.tiles = (int)tiles; P.chunks = chunks;
            P.x_bytes = (unsigned)x_bytes; P.w_bytes = (unsigned)w_bytes;
            for (int t = 0; t < kTaps; ++t) P.tap_off[t] = (int)(16 * ((t / s.S) * IW + t % s.S) * s.dil);
            P.by_px_tiles = make_fastdiv((int)px_tiles); P.by_tiles_y = make_fastdiv(tiles_y);
            P.by_cells_img = make_fastdiv(P.cells_img); P.by_IW = make_fastdiv(P.IW);
            P.by_thwo = make_fastdiv(TH * s.Wo); P.by_Wo = make_fastdiv(s.Wo);
        }
    };
    for (int NI = 2; NI <= s.N && (int64_t)NI * s.Ho * s.Wo <= 512; ++NI) consider(NI, 1);
    for (int TH = std::min(s.Ho, 512 / s.Wo), last = 0; TH >= 1; --TH) {        // (tiles of at most 512 pixels, however tall the image)
        const int tiles_y = (s.Ho + TH - 1) / TH;
        if (tiles_y != last) consider(1, tiles_y);
        last = tiles_y;
    }
    return best;
}

SplitPlan plan_split(const Conv2dShape& s)
{
    thread_local PlanCache<SplitPlan> cache;
    return cache.get(s, 0, [&] { return search_split(s); });
}

template <int PH, int PB>
hipError_t launch_one(const float* x, const float* w, float* y, const SplitPlan& a, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_f32_split_kernel<PH, PB>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes(PH));
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel("mfma_f32_split_kernel", 10 * PH + PB, a.P.NI, a.P.TH), (mfma_f32_split_kernel<PH, PB>),
                    dim3(a.grid), dim3(64 * (mul_waves(PH) + PH + win_waves(PH))), lds_bytes(PH), st, x, w, y, a.P);
    return hipGetLastError();
}

}  // namespace

bool mfma_f32_split_supported(const Conv2dShape& s) { return plan_split(s).ok; }

// (the plan's ticks, fitted to 81 launches)
double mfma_f32_split_estimate(const Conv2dShape& s) { return 3.62e-4 * plan_split(s).est + 1.06; }

hipError_t launch_mfma_f32_split(const float* x, const float* w, float* y, const Conv2dShape& s, hipStream_t st, const Epilogue& ep)
{
    SplitPlan a = plan_split(s);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
    switch (10 * a.PH + a.PB) {
        case 11: return launch_one<1, 1>(x, w, y, a, st);
        case 12: return launch_one<1, 2>(x, w, y, a, st);
        case 21: return launch_one<2, 1>(x, w, y, a, st);
        default: return launch_one<4, 1>(x, w, y, a, st);
    }
}

}  // namespace swconv
