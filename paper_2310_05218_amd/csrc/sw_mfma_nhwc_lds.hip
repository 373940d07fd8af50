// Multi-channel convolution on channel-last tensors (fp32, bf16, IEEE half or int8) with both operands in LDS, the window brought
// in by direct-to-LDS loads (paper, section 3: every tap a small matrix product whose shift is an address; section 1.1:
// reduced precision on the same sliding sums).
//
//   x [N, H, W, C]     w [C_out, R, S, C]     y [N, H_out, W_out, C_out]     fp32 values or 16-bit patterns, fp32 sums
//
// The kernels that read their pixel operands straight from global memory (sw_mfma_bf16_nhwc.hip) or copy the window
// through registers (sw_mfma_nhwc.hip) are bound by cache-line look-ups and by the copy.  Here a load instruction takes
// whole lines: the rectangle of input pixels a tile touches (its window, padding included as out-of-range addresses that
// arrive as zeros) goes to LDS in 16-byte pieces (8 channels, fp32: 4), 64 consecutive pieces per instruction, and a lane's
// pixel operand for (pixel, tap, step) is one 16-byte LDS read at cell(pixel) + (r IW + s) dilation: the eight channels of
// its half of a v_mfma_f32_32x32x16_{bf16,f16}, or the four channels that four v_mfma_f32_32x32x2_f32 take one by one (K
// index j of lane half kq = channel 4 kq + j of the step's eight: the matrix instruction does not care which channel a K
// index stands for as long as both operands agree).  A cell's NP pieces are stored at slot = piece ^ key, key = the cell's
// 256-byte row of LDS modulo NP, which spreads the 16 cells a read serves per pass over all 64 banks whatever NP is (a
// 16-byte read is served 16 consecutive lanes at a time: measured, two lanes on one bank collide if and only if their numbers
// differ in the low four bits only).
//
// Workgroup = 32 CB output channels, persistent: it fetches the filters of its channels once ([channel][tap][C] rows as
// they lie in w, odd row pitch in pieces) and then walks over tiles of up to 128 PB output pixels (rows of one image, or
// whole small images), the window of the next (tile, chunk of channels) in flight while this one multiplies: four
// wavefronts only load, four multiply (pixel block 4b + w to wavefront w, all channel blocks).  Filters are the A operand,
// pixels the B operand: a lane of the result holds, for its pixel, groups of four consecutive output channels (fp32: one
// 16-byte store; 16-bit and int8 results: 8 and 4 bytes, which the lane halves exchange (v_permlane32_swap) for whole 16-byte pieces
// where C_out allows).
//
// int8 (x, w int8; exact int32 sums): a piece is 16 channels, a step of two pieces one v_mfma_i32_32x32x32_i8.  The sums
// leave as int32 (16-byte stores, like fp32) or requantised to int8, q = clamp(rne(scale * float(sum + bias))).  Biases and scales
// are read from LDS.
//
// Filters too large to stay in LDS whole (16-bit: 3 x 3 from 144 input channels on at 64 output channels per workgroup;
// fp32: from 72 on) travel with the window instead: every stage carries the chunk's part of the filters,
// [channel][tap][NP pieces] at an odd row pitch, fetched by the same loaders from L2 again for every tile.  The multipliers
// read them at the stage's address; all else is the same code (FS, a compile-time switch, so that the resident form pays
// nothing for it).
//
// What bounds it (time stamps of 64 -> 64 at 56 x 56, bf16, 32 images: two tiles of two chunks a workgroup; cycles): 6.3 k until the
// first chunk is multiplied, of which 1.2 k are the first scalar loads and 2.4 k the filters' loads (73 KB at 31 bytes a cycle and CU); 3.4 k a
// chunk for 2.3 k of matrix instructions; 2.5 k of stores a tile.  An operand read and a matrix instruction take turns in each wavefront's
// issue, so the loop is written for that: reads between the matrix instructions (they were issued in a block before them and waited for,
// because a branch stood around them: 4.65 k a chunk), a tap's bookkeeping in eight scalar instructions, addresses in four vector
// ones.  Before and after, us (replayed graphs of ten, batch 32): this layer 18.4 -> 15.5, 128 -> 128 at 28 x 28 int8 12.3 -> 10.8, 256 -> 256 at
// 14 x 14 bf16 18.3 -> 15.2, 256 -> 64 at 56 x 56 1 x 1 bf16 17.7 -> 13.8, fp32 55.7 -> 45.7; 8 x 272 -> 80 at 37 x 8 bf16 23.9 -> 15.1,
// 5 x 320 -> 416 at 7 x 7 5 x 5 stride 2 47.5 -> 28.7; 220 layers of all formats 1.20 on the average, none slower.
// Tried and not kept: the products of a pixel block in two halves on two wavefronts of a SIMD (3.0 k a chunk, but 2.4 k more a tile for the
// halves to meet: 18.4); all eight wavefronts loading and multiplying in turn (20.4).
#include <algorithm>
#include <type_traits>

#include "swconv_internal.h"

namespace swconv {

namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef int intx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8 __attribute__((ext_vector_type(8)));

#define SW_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr size_t kLdsTotal = 156 * 1024;       // two stages and what the search leaves beside them
constexpr size_t kLdsAll = 160 * 1024;
constexpr size_t kFilterMax = 76 * 1024;       // resident filters of a workgroup
constexpr int kMaxWK = 12;                     // window loads per loading wavefront and stage
constexpr int kMaxFK = 12;                     // filter loads per loading wavefront and stage (filters fetched per chunk)
constexpr unsigned kBeyond = 0x80000000u;      // a byte offset no x or w of less than 2 GiB reaches
constexpr unsigned kBeyondY = 0xffff0000u;     // ... and no tile of y: 256 pixels of 65535 blocks of 64 channels of four bytes
// formats beyond Elem's: int8 operands with exact int32 sums, leaving as int32 or requantised to int8
constexpr int kFmtS8 = 3, kFmtS8Q = 4, kFormats = 5;

struct LdsParams {
    Epilogue ep;
    Requant rq;                    // (int8 -> int8)
    int rq_off;                    // 32 CB biases, then (int8 -> int8) 32 CB scales, once per workgroup
    int N, H, W, C, C_out, R, S, stride, pad, dil, Ho, Wo;
    int pix_bytes, cpt;            // bytes of a pixel's channels; 16-byte pieces of a tap in a filter row (C / 8, fp32: C / 4)
    int NI, TH, tiles_y, tiles;    // images and output rows per tile, row tiles per image, tiles in all
    int IH, IW, cells_img, WC;     // window rows and columns of one image, their product, cells of a window
    int NP, chunks;                // 16-byte pieces per pixel and chunk (2, 4 or 8), chunks of 8 NP channels
    int wloads;                    // 64-piece loads per window stage
    int frow, fpitch;              // 16-byte pieces of an output channel's filters (R S C / 8), row pitch in LDS (odd)
    int win_off, stage_bytes;      // window stages behind the filters
    int fstream;                   // the filters do not fit LDS whole: the chunk's part ([channel][tap][NP pieces], pitch fp2)
    int fp2, fs_off, fsloads;      // travels with every window stage, fs_off bytes behind the window, in fsloads loads
    int wide_out;                  // y is made of whole 16-byte pieces
    int stages;                    // window stages: two, or three where LDS has room
    // from a loading lane's cell to that of its next load, 256 / NP cells on: images, rows and columns of the window, and bytes of x; what the
    // end of a window row and the end of an image add to the bytes
    int d_img, d_row, d_col, d_bytes, row_bytes, img_bytes;
    int d_co, d_piece;             // from a lane's filter piece to that of its next load, 256 pieces on: output channels, pieces
    unsigned x_bytes, w_bytes;
    FastDiv by_tiles_y, by_cells_img, by_IW, by_thwo, by_Wo, by_fpitch, by_fp2;
};

__device__ __forceinline__ unsigned round16_pair(float a, float b, bool f16)       // nearest even
{
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
    const floatx2 v = {a, b};
    return f16 ? __builtin_bit_cast(unsigned, __builtin_convertvector(v, halfx2)) : __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// s_waitcnt vmcnt for at most n operations in flight (or the next smaller count that there is an instruction for here)
template <int n>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory"); }
__device__ __forceinline__ void wait_loads_but(int n)
{
    if (n >= 8) {
        if (n >= 16) wait_loads<16>();
        else if (n >= 12) wait_loads<12>();
        else if (n >= 10) wait_loads<10>();
        else wait_loads<8>();
    } else if (n >= 4) {
        if (n >= 6) wait_loads<6>();
        else if (n == 5) wait_loads<5>();
        else wait_loads<4>();
    } else {
        if (n == 3) wait_loads<3>();
        else if (n == 2) wait_loads<2>();
        else if (n == 1) wait_loads<1>();
        else wait_loads<0>();
    }
}

// barrier without the fence of __syncthreads (which would wait for the loads and stores in flight)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// EK: format (Elem: fp32, bf16, IEEE half; kFmtS8, kFmtS8Q).  CB: blocks of 32 output channels per workgroup.  PB: blocks of 32 pixels per wavefront.
// KSC: steps of 16 channels per tap and chunk (NP / 2).  FS: filters per chunk with the window (else resident).  ONE: a single tap.
template <int EK, int CB, int PB, int KSC, bool FS, bool ONE>
__global__ __launch_bounds__(512, 2) void mfma_nhwc_lds_kernel(const unsigned char* __restrict__ x, const unsigned char* __restrict__ w,
                                                               unsigned char* __restrict__ yb, const LdsParams P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr bool F16 = EK == kElemF16;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int co0 = blockIdx.y * (32 * CB);
    const int steps_per_wg = ((P.tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x) * P.chunks;   // (tile, chunk) steps
    const int m = P.NP - 1, lnp = __builtin_ctz(P.NP);

    if (wave >= 4) {
        // ---------------------------------------------------------------------------------------- the loaders
        const int lw = wave - 4;
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(w), 0, P.w_bytes, 0x00020000);
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(x), 0, P.x_bytes, 0x00020000);
        // this lane's slot in each window load of this wavefront (loads lw, lw + 4, ...): its cell's place in the window
        // (image, row, column) and the byte offset of its piece from the tile's origin; what changes per tile is the
        // origin and which rows and images exist
        // (in steps from load to load: with the divisions for each the first load left 1.5 k cycles later)
        int wrow[kMaxWK], wimg[kMaxWK];
        unsigned wofs[kMaxWK];
        {
            const int q = 64 * lw + lane;
            int cell = q >> lnp;                                    // (NP is a power of two)
            const int piece = (q & m) ^ ((cell >> (4 - lnp)) & m);  // (the same in all of a lane's loads: they are 16 rows of 256 bytes apart)
            int i = fast_div(cell, P.by_cells_img), rem = cell - i * P.cells_img;
            int e = fast_div(rem, P.by_IW), f = rem - e * P.IW;
            unsigned ofs = (unsigned)(((i * P.H + e) * P.W + f - P.pad) * P.pix_bytes + 16 * piece);
#pragma unroll
            for (int k = 0; k < kMaxWK; ++k) {
                if (lw + 4 * k >= P.wloads) break;
                const bool in = cell < P.WC && (unsigned)(f - P.pad) < (unsigned)P.W;
                wimg[k] = i;
                wrow[k] = in ? e : -(1 << 20);                      // (a row that never exists)
                wofs[k] = ofs;
                cell += 256 >> lnp;
                i += P.d_img; e += P.d_row; f += P.d_col; ofs += P.d_bytes;
                if (f >= P.IW) { f -= P.IW; ++e; ofs += P.row_bytes; }
                if (e >= P.IH) { e -= P.IH; ++i; ofs += P.img_bytes; }
            }
        }
        // (filters per chunk) this lane's slot in each filter load of this wavefront: piece j % NP of tap j / NP of output
        // channel co, j = q % fp2; byte offset in w for chunk 0
        unsigned fofs[kMaxFK];
#pragma unroll
        for (int k = 0; k < kMaxFK; ++k) {
            fofs[k] = kBeyond;
            if (FS && lw + 4 * k < P.fsloads) {
                const int q = 64 * (lw + 4 * k) + lane;
                const int co = fast_div(q, P.by_fp2), j = q - co * P.fp2;
                const int tap = j >> lnp, piece = j & m;
                if (co < 32 * CB && tap < P.R * P.S && co0 + co < P.C_out)
                    fofs[k] = (unsigned)(((co0 + co) * P.R * P.S + tap) * P.pix_bytes + 16 * piece);
            }
        }
        int l_tile = blockIdx.x, l_ch = 0, l_stage = 0;             // the next step to load
        auto issue = [&]() __attribute__((always_inline)) {
            const int ig = fast_div(l_tile, P.by_tiles_y), ty = l_tile - ig * P.tiles_y;
            const int n0 = ig * P.NI, gr0 = ty * P.TH * P.stride - P.pad;
            const unsigned origin = (unsigned)((n0 * P.H + gr0) * P.W * P.pix_bytes + l_ch * (16 * P.NP));
            unsigned char* sw = smem + P.win_off + l_stage * P.stage_bytes;
#pragma unroll
            for (int k = 0; k < kMaxWK; ++k) {
                if (lw + 4 * k >= P.wloads) break;
                const bool in = (unsigned)(gr0 + wrow[k]) < (unsigned)P.H && n0 + wimg[k] < P.N;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, SW_LDS_PTR(sw + 1024 * (lw + 4 * k)), 16, in ? origin + wofs[k] : kBeyond, 0, 0, 0);
            }
            if (FS) {
                const unsigned choff = (unsigned)(l_ch * (16 * P.NP));
#pragma unroll
                for (int k = 0; k < kMaxFK; ++k) {
                    if (lw + 4 * k >= P.fsloads) break;
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, SW_LDS_PTR(sw + P.fs_off + 1024 * (lw + 4 * k)), 16,
                                                             fofs[k] == kBeyond ? kBeyond : fofs[k] + choff, 0, 0, 0);
                }
            }
            if (++l_ch == P.chunks) { l_ch = 0; l_tile += gridDim.x; }
            if (++l_stage == P.stages) l_stage = 0;
        };
        const int stage_loads = max(0, (P.wloads - lw + 3) >> 2) + (FS ? max(0, (P.fsloads - lw + 3) >> 2) : 0);
        const int ahead = P.stages - 1;
#pragma unroll 1
        for (int s = 0; s < min(ahead, steps_per_wg); ++s) issue();
#pragma unroll 1
        for (int s = 0; s < steps_per_wg; ++s) {
            // this wavefront's loads of step s have landed; behind them are those of step s + 1, where there is a third stage
            wait_loads_but(ahead == 2 && s + 1 < steps_per_wg ? stage_loads : 0);
            lds_barrier();                              // barrier s: step s is complete, step s - 1 has been multiplied
            if (s + ahead < steps_per_wg) issue();
        }
        wait_loads_but(0);
        return;
    }

    // -------------------------------------------------------------------------------------------- the multipliers
    // the filters, once: slot q of the filter area is piece q % fpitch of output channel q / fpitch
    if (!FS) {
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(w), 0, P.w_bytes, 0x00020000);
        int co = fast_div(tid, P.by_fpitch), j = tid - co * P.fpitch;
        unsigned off = (unsigned)(((co0 + co) * P.frow + j) * 16);
        const unsigned step = (unsigned)((P.d_co * P.frow + P.d_piece) * 16), turn = (unsigned)((P.frow - P.fpitch) * 16);
        const int co_end = min(32 * CB, P.C_out - co0);
#pragma unroll 1
        for (int k = 1024 * wave; k < 32 * CB * 16 * P.fpitch; k += 4096) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, SW_LDS_PTR(smem + k), 16, co < co_end && j < P.frow ? off : kBeyond, 0, 0, 0);
            co += P.d_co; j += P.d_piece; off += step;
            if (j >= P.fpitch) { j -= P.fpitch; ++co; off += turn; }
        }
    }
    // the workgroup's biases (requantisation: and scales) to LDS (the first barrier orders them before their use)
    if (tid < 32 * CB) {
        const int co = co0 + tid;
        if constexpr (EK == kFmtS8Q) {
            reinterpret_cast<int*>(smem + P.rq_off)[tid] = (P.rq.bias != nullptr && co < P.C_out) ? P.rq.bias[co] : 0;
            reinterpret_cast<float*>(smem + P.rq_off)[32 * CB + tid] = co < P.C_out ? P.rq.scale[co] : 0.f;
        } else if constexpr (EK != kFmtS8) {
            reinterpret_cast<float*>(smem + P.rq_off)[tid] = (P.ep.bias != nullptr && co < P.C_out) ? P.ep.bias[co] : 0.f;
        }
    }
    const int lj = lane & 31, kq = lane >> 5;
    const int thwo = P.TH * P.Wo, HoWo = P.Ho * P.Wo;
    // this wavefront's pixel blocks: block 4b + wave of the tile; the pixel's cell in the window does not depend on the tile
    int cell0[PB];                                                         // (in bytes)
#pragma unroll
    for (int b = 0; b < PB; ++b) {
        const int p = 32 * (4 * b + wave) + lj;
        const int pc = p < P.NI * thwo ? p : 0;
        const int i = fast_div(pc, P.by_thwo), rem = pc - i * thwo;
        const int ol = fast_div(rem, P.by_Wo), ow = rem - ol * P.Wo;
        cell0[b] = (i * P.cells_img + (ol * P.IW + ow) * P.stride) << (lnp + 4);
    }
    // A operand of (channel block cb, tap, step ks): resident filters: row pitch fpitch pieces, C / 8 pieces per tap, the
    // chunk's NP pieces at chunk NP; filters per chunk: row pitch fp2, NP pieces per tap
    const int apitch = FS ? P.fp2 : P.fpitch, cpt = FS ? P.NP : P.cpt;
    const unsigned char* arow = smem + (lj * apitch + kq) * 16;            // + 32 cb apitch 16 + (tap cpt + 2 ks) 16

    // (the rectifier as a lower bound; without one a NaN, which the maximum with a number ignores and that with a NaN keeps)
    const float floor_ = P.ep.relu ? 0.f : __builtin_nanf("");

    using Acc = std::conditional_t<(EK >= kFmtS8), intx16, floatx16>;
    Acc acc[CB][PB];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int b = 0; b < PB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[cb][b][v] = 0;
    };
    const int taps = ONE ? 1 : P.R * P.S;
    const int tap_bytes = cpt * 16, last_at = (taps - 1) * tap_bytes;
    // bytes in the window from a tap to the next of its row, to the first of the next row, to the last
    const int cshift = lnp + 4, step_col = P.dil << cshift, step_row = ((P.IW - P.S + 1) * P.dil) << cshift;
    const int last_tap = (((P.R - 1) * P.IW + P.S - 1) * P.dil) << cshift;
    int tile = blockIdx.x, ch = 0, stage = 0;
    __builtin_amdgcn_s_waitcnt(0);                                         // (this wavefront's share of the filters)
#pragma unroll 1
    for (int s = 0; s < steps_per_wg; ++s) {
        // barrier s, without the fence of __syncthreads: that would wait for the stores of the tile before to be
        // acknowledged (about 2 us per tile); nothing here reads what they wrote
        lds_barrier();
        if (ch == 0) {
            asm volatile("");                                              // (a branch, not a select in each register for every chunk)
            clear();
        }
        const unsigned char* sw = smem + P.win_off + stage * P.stage_bytes;
        const unsigned char* ab = FS ? arow + P.win_off + stage * P.stage_bytes + P.fs_off : arow + (ch * P.NP) * 16;
        if (++stage == P.stages) stage = 0;
        // One step (16 channels of a tap) at a time: CB PB matrix instructions on CB + PB operand reads.  The reads of step t + D - 1
        // sit between the matrix instructions of step t, in no branch: where paths with and without reads meet, the compiler waits as
        // if there were none.  D (a multiple of KSC): a read takes some 200 to 300 cycles to arrive, a matrix instruction 32.
        constexpr int D = EK == kElemF32 ? (KSC > 2 ? KSC : 2) : CB * PB == 4 ? 4 : CB * PB == 1 || KSC == 4 ? 8 : 6;
        struct Ops {
            intx4 a[CB], b[PB];
        };
        Ops ops[D];
        int sc = 0, at = 0, toff = 0;                                      // the next tap: its column, its place in the filters and in the window
        int cell[PB], swizzle[PB];
        auto read_step = [&](Ops& o, int ks) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) o.a[cb] = *reinterpret_cast<const intx4*>(ab + at + (32 * cb * apitch + 2 * ks) * 16);
#pragma unroll
            for (int b = 0; b < PB; ++b) {
                if (ks == 0) {
                    cell[b] = cell0[b] + toff;
                    swizzle[b] = (cell[b] >> 4) & (m << 4);
                }
                o.b[b] = *reinterpret_cast<const intx4*>(sw + cell[b] + (swizzle[b] ^ ((2 * ks + kq) << 4)));
            }
            if (ks == KSC - 1) {
                // (past the last tap: the last once more)
                at = min(at + tap_bytes, last_at);
                const bool turn = ++sc == P.S;
                toff = min(toff + (turn ? step_row : step_col), last_tap);
                sc = turn ? 0 : sc;
            }
        };
        auto multiply_step = [&](const Ops& o) __attribute__((always_inline)) {
            if constexpr (EK == kElemF32) {
                // a piece is four channels: matrix instruction j of the step takes channel j of the two lane halves' pieces
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int b = 0; b < PB; ++b)
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb) {
                            // (the whole vector is cast, then indexed: a cast of one indexed element took element 0)
                            const floatx4 af = __builtin_bit_cast(floatx4, o.a[cb]), bf = __builtin_bit_cast(floatx4, o.b[b]);
                            acc[cb][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[j], bf[j], acc[cb][b], 0, 0, 0);
                        }
            } else {
#pragma unroll
                for (int b = 0; b < PB; ++b)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        if constexpr (EK >= kFmtS8)
                            acc[cb][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(o.a[cb], o.b[b], acc[cb][b], 0, 0, 0);
                        else if constexpr (F16)
                            acc[cb][b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(halfx8, o.a[cb]),
                                                                                __builtin_bit_cast(halfx8, o.b[b]), acc[cb][b], 0, 0, 0);
                        else
                            acc[cb][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, o.a[cb]),
                                                                                 __builtin_bit_cast(bf16x8, o.b[b]), acc[cb][b], 0, 0, 0);
                    }
            }
        };
        auto interleave = [&]() __attribute__((always_inline)) {
            constexpr int M = CB * PB * (EK == kElemF32 ? 4 : 1), RD = CB + PB;
#pragma unroll
            for (int i = 0; i < M; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (RD * (i + 1) / M > RD * i / M) {
                    __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                    if constexpr (RD > M) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    else __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                }
            }
        };
        if constexpr (ONE) {
#pragma unroll
            for (int ks = 0; ks < KSC; ++ks) read_step(ops[ks], ks);
#pragma unroll
            for (int ks = 0; ks < KSC; ++ks) multiply_step(ops[ks]);
        } else {
            const int steps = taps * KSC;
#pragma unroll
            for (int d = 0; d < D - 1; ++d) read_step(ops[d], d % KSC);
            int t = 0;
#pragma unroll 1
            for (; t + D <= steps; t += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    __builtin_amdgcn_sched_barrier(0);
                    read_step(ops[(d + D - 1) % D], (d + D - 1) % KSC);
                    multiply_step(ops[d]);
                    interleave();
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int d = 0; d < D - 1; ++d)
                if (t + d < steps) multiply_step(ops[d]);
        }

        if (++ch < P.chunks) continue;
        ch = 0;
        // ---- the tile is finished: register v of a lane is output channel 8 (v / 4) + 4 kq + v % 4 of the block
        const int ig = fast_div(tile, P.by_tiles_y), ty = tile - ig * P.tiles_y;
        const int n0 = ig * P.NI, row0 = ty * P.TH;
        tile += gridDim.x;
        const int valid_px = P.NI > 1 ? min(P.NI, P.N - n0) * HoWo : min(P.TH, P.Ho - row0) * P.Wo;
        constexpr int OB = EK == kFmtS8Q ? 1 : (EK == kElemF32 || EK == kFmtS8) ? 4 : 2;
        // (a tile's pixels are consecutive in y.  Stores by offsets from the tile: pixels beyond it fall out of the buffer's range, channels
        // beyond the last are given such an offset, and no store needs a branch)
        const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(
            yb + (((int64_t)n0 * HoWo + row0 * P.Wo) * P.C_out + co0) * OB, 0, (unsigned)(valid_px * P.C_out - co0) * OB, 0x00020000);
        const int co_end = P.C_out - co0;
        const unsigned char* const lb = smem + P.rq_off + 16 * kq;         // biases and scales of the lane's channels
        if constexpr (OB == 4) {
            // four consecutive output channels of a pixel are 16 bytes: stored as they lie in the accumulators
#pragma unroll
            for (int b = 0; b < PB; ++b) {
                const unsigned off = (unsigned)((32 * (4 * b + wave) + lj) * P.C_out + 4 * kq) * 4;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int c = cb * 32 + 8 * q;
                        intx4 v;
                        if constexpr (EK == kFmtS8) {
#pragma unroll
                            for (int j = 0; j < 4; ++j) v[j] = acc[cb][b][4 * q + j];
                        } else {
                            const floatx4 bias = *reinterpret_cast<const floatx4*>(lb + 4 * c);
                            floatx4 f;
#pragma unroll
                            for (int j = 0; j < 4; ++j) f[j] = fmaxf(acc[cb][b][4 * q + j] + bias[j], floor_);
                            v = __builtin_bit_cast(intx4, f);
                        }
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, v), yr, c + 4 * kq < co_end ? off + 4 * c : kBeyondY, 0, 0);
                    }
            }
        } else {
            // 16-bit and requantised int8 results: four consecutive output channels of a lane are 4 OB bytes
            using Pack = std::conditional_t<EK == kFmtS8Q, int, intx2>;
            // (int8: a copy with the rectifier and one without, one of which runs, in place of a select in every result)
#pragma unroll
            for (int relu = 0; relu < (EK == kFmtS8Q ? 2 : 1); ++relu) {
                if (EK == kFmtS8Q && relu != (P.rq.relu != 0)) continue;
                auto pack = [&](int cb, int b, int q) __attribute__((always_inline)) {
                    const int c = cb * 32 + 8 * q;
                    if constexpr (EK == kFmtS8Q) {
                        // q = clamp(rne(scale * float(acc + bias)), relu ? 0 : -128, 127), every step in fp32 as the definition has it
                        const intx4 qb = *reinterpret_cast<const intx4*>(lb + 4 * c);
                        const floatx4 qs = *reinterpret_cast<const floatx4*>(lb + 4 * (32 * CB + c));
                        const int t0 = (int)acc[cb][b][4 * q] + qb[0], t1 = (int)acc[cb][b][4 * q + 1] + qb[1];
                        const int t2 = (int)acc[cb][b][4 * q + 2] + qb[2], t3 = (int)acc[cb][b][4 * q + 3] + qb[3];
                        return relu ? requant_pack4<true>(t0, t1, t2, t3, qs[0], qs[1], qs[2], qs[3]) : requant_pack4<false>(t0, t1, t2, t3, qs[0], qs[1], qs[2], qs[3]);
                    } else {
                        const floatx4 bias = *reinterpret_cast<const floatx4*>(lb + 4 * c);
                        float v[4];
#pragma unroll
                        for (int j = 0; j < 4; ++j) v[j] = fmaxf(acc[cb][b][4 * q + j] + bias[j], floor_);
                        return intx2{(int)round16_pair(v[0], v[1], F16), (int)round16_pair(v[2], v[3], F16)};
                    }
                };
#pragma unroll
                for (int b = 0; b < PB; ++b) {
                    if (32 * (4 * b + wave) >= valid_px) continue;                     // (wave-uniform)
                    const unsigned off = (unsigned)((32 * (4 * b + wave) + lj) * P.C_out) * OB;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        Pack v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] = pack(cb, b, q);
                        if (P.wide_out) {
                            // the lane halves swap registers, so that a lane holds 16 consecutive bytes of its pixel
                            if constexpr (OB == 2) {
                                // (channels 8 kq .. 8 kq + 7 of each half block)
#pragma unroll
                                for (int h = 0; h < 2; ++h) {
                                    const auto r0 = __builtin_amdgcn_permlane32_swap(v[2 * h][0], v[2 * h + 1][0], false, false);
                                    const auto r1 = __builtin_amdgcn_permlane32_swap(v[2 * h][1], v[2 * h + 1][1], false, false);
                                    const int c = cb * 32 + 16 * h + 8 * kq;
                                    __builtin_amdgcn_raw_buffer_store_b128(uintx4{r0[0], r1[0], r0[1], r1[1]}, yr, c < co_end ? off + 2 * c : kBeyondY, 0, 0);
                                }
                            } else {
                                // (channels 16 kq .. 16 kq + 15)
                                const auto r0 = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
                                const auto r1 = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
                                const int c = cb * 32 + 16 * kq;
                                __builtin_amdgcn_raw_buffer_store_b128(uintx4{r0[0], r0[1], r1[0], r1[1]}, yr, c < co_end ? off + c : kBeyondY, 0, 0);
                            }
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const int c = cb * 32 + 8 * q + 4 * kq;
                                const unsigned at = c < co_end ? off + c * OB : kBeyondY;
                                if constexpr (OB == 2) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v[q]), yr, at, 0, 0);
                                else __builtin_amdgcn_raw_buffer_store_b32((unsigned)v[q], yr, at, 0, 0);
                            }
                        }
                    }
                }
            }
        }
    }
}

struct LdsPlan {
    bool ok = false;
    int CB = 0, PB = 0;
    size_t lds = 0;
    unsigned gx = 0, gy = 0;
    double est = 0;
    int64_t tiles = 0;
    LdsParams P;
};

LdsPlan search_plan(const Conv2dShape& s, int ek, const void* x, const void* w, const void* y)
{
    LdsPlan best;
    const int RS = s.R * s.S;
    const int es = ek >= kFmtS8 ? 1 : (int)elem_size(ek), cpp = 16 / es;    // bytes of an element, channels in a 16-byte piece
    const int ob = ek == kFmtS8 ? 4 : ek == kFmtS8Q ? 1 : es;                // bytes of an output element
    const int64_t x_bytes = (int64_t)s.N * s.H * s.W * s.C_in * es, w_bytes = (int64_t)s.C_out * RS * s.C_in * es;
    // a step of the matrix instructions takes two pieces; a lane stores four consecutive output channels at once
    if (s.C_in % (2 * cpp) != 0 || s.C_out % 4 != 0 || x_bytes >= (1LL << 31) || w_bytes >= (1LL << 31)) return best;
    if (reinterpret_cast<uintptr_t>(x) % 16 != 0 || reinterpret_cast<uintptr_t>(w) % 16 != 0 ||
        reinterpret_cast<uintptr_t>(y) % (4 * ob) != 0)
        return best;
    if ((int64_t)s.N * s.Ho * s.Wo * s.C_out >= (1LL << 40)) return best;
    const int frow = RS * s.C_in / cpp, fpitch = frow | 1;
    const int64_t IW = (int64_t)(s.Wo - 1) * s.stride + (int64_t)(s.S - 1) * s.dil + 1;
    const int HoWo = s.Ho * s.Wo;
    // lane halves exchange their results where y is made of whole 16-byte pieces
    const bool wide_out = ob <= 2 && s.C_out % (16 / ob) == 0 && reinterpret_cast<uintptr_t>(y) % 16 == 0;
    // CB blocks of 32 output channels per workgroup; filters resident (fstream = false) or fetched per chunk with the window;
    // NP pieces of eight channels per pixel and chunk: the wider the chunk, the fewer steps; the narrower, the larger the
    // tile LDS holds
    auto consider = [&](int CB, bool fstream, int PB, int NP, int NI, int tiles_y) {
        if (s.C_in % (cpp * NP) != 0) return;
        const int chunks = s.C_in / (cpp * NP);
        const int co_blocks = (s.C_out + 32 * CB - 1) / (32 * CB);
        if (co_blocks > 65535) return;
        const int fp2 = (RS * NP) | 1;
        const int64_t fsloads = fstream ? ((int64_t)32 * CB * fp2 + 63) / 64 : 0;
        if (fsloads > 4 * kMaxFK) return;
        const size_t fbytes = fstream ? 0 : ((size_t)32 * CB * fpitch * 16 + 1023) & ~(size_t)1023;
        if (fbytes > kFilterMax) return;
        // Beside the stages only the biases and scales are allocated (512 bytes).  The search leaves more: room that results in LDS once took, which
        // the estimates below were fitted with.  Without it 291 of 20000 drawn layers get larger tiles of two stages in place of three, 0.66 to 1.8 of
        // them, 0.957 in the median, as fast (640 -> 48 at 114 x 114 2 x 2 dilation 2, 7 images bf16 54 / 82 us, 608 -> 624 at 10 x 78 3x3 dilation 2,
        // 8 images half 65 / 36).
        const size_t beside = (wide_out ? (size_t)4 * 32 * (32 * CB * ob + 16) : 0) + (ek == kFmtS8Q ? 512 : 0);
        const int tp_max = 128 * PB;
        const int TH = (s.Ho + tiles_y - 1) / tiles_y;
        if ((int64_t)TH * s.Wo * NI > tp_max || (s.Ho + TH - 1) / TH != tiles_y) return;
        const int64_t IH = (int64_t)(TH - 1) * s.stride + (int64_t)(s.R - 1) * s.dil + 1;
        const int64_t WC = NI * IH * IW;
        const int64_t wloads = (WC * NP + 63) / 64;
        if (wloads > 4 * kMaxWK) return;
        const size_t stage = (size_t)(wloads + fsloads) * 1024;
        const size_t lds = fbytes + 2 * stage + beside;
        if (lds > kLdsTotal) return;
        const int64_t groups = (s.N + NI - 1) / NI;
        const int64_t tiles = groups * tiles_y;
        if (tiles > 2147483647LL) return;
        double est;
        if (es == 4) {
            // fp32: the matrix instructions bound a step (64 cycles each, four per 16-byte operand pair) unless its loads
            // take longer (about 10 bytes per clock and CU out of L2, 5 for a single tap, whose pixels come from memory
            // once); a step costs about 1500 cycles beyond them (pipeline fill, barrier), a tile its stores.  Cycles of a
            // workgroup: its tiles one after the other; more workgroups than CUs run in turns.
            const double mfma = (double)RS * (NP / 2) * 4 * CB * PB * 64;
            const double load = (double)stage / (RS == 1 ? 5.0 : 10.0);
            const double tile_cycles = chunks * (std::max(mfma + 700, load) + 800) + 900.0 * CB * PB;
            const int64_t gx = std::max<int64_t>(1, std::min<int64_t>(tiles, 256 / std::min(co_blocks, 256)));
            const double turns = std::max(1.0, (double)gx * co_blocks / 256.0);
            est = turns * (double)((tiles + gx - 1) / gx) * tile_cycles + (double)fbytes / 13.0;
        } else {
            // 16-bit: LDS operand reads bound a step.  Periods of one block through all of K: every wavefront multiplies PB
            // blocks, live or not; 256 workgroups at a time.  Two blocks per wavefront halve the filter reads per matrix
            // instruction, but with a single tap a step is too short for them to pay (measured); one channel block per
            // workgroup doubles the window reads per matrix instruction; filters per chunk are fetched again for every tile.
            est = std::max((double)PB, (double)tiles * co_blocks * PB / 256.0) * (PB == 2 ? (RS >= 4 ? 0.8 : 1.1) : 1.0) *
                  (1.0 + 0.05 * (chunks - 1)) * (CB == 1 && s.C_out > 32 ? 1.2 : 1.0) * (fstream ? 1.3 : 1.0);
        }
        if (best.ok && (est > best.est || (est == best.est && tiles >= best.tiles))) return;
        best.ok = true;
        best.CB = CB;
        best.PB = PB;
        best.est = est;
        best.tiles = tiles;
        best.gy = (unsigned)co_blocks;
        best.gx = (unsigned)std::max<int64_t>(1, std::min<int64_t>(tiles, 256 / std::min(co_blocks, 256)));
        LdsParams& P = best.P;
        P.N = s.N; P.H = s.H; P.W = s.W; P.C = s.C_in; P.C_out = s.C_out; P.R = s.R; P.S = s.S; P.stride = s.stride;
        P.pad = s.pad; P.dil = s.dil; P.Ho = s.Ho; P.Wo = s.Wo;
        P.pix_bytes = s.C_in * es; P.cpt = s.C_in / cpp;
        P.NI = NI; P.TH = TH; P.tiles_y = tiles_y; P.tiles = (int)tiles;
        P.IH = (int)IH; P.IW = (int)IW; P.cells_img = (int)(IH * IW); P.WC = (int)WC;
        P.NP = NP; P.chunks = chunks; P.wloads = (int)wloads;
        P.frow = frow; P.fpitch = fpitch;
        P.fstream = fstream ? 1 : 0; P.fp2 = fp2; P.fs_off = (int)(wloads * 1024); P.fsloads = (int)fsloads;
        P.win_off = (int)fbytes; P.stage_bytes = (int)stage;
        P.wide_out = wide_out ? 1 : 0;
        P.stages = 2;
        P.x_bytes = (unsigned)x_bytes; P.w_bytes = (unsigned)w_bytes;
        const int dc = 256 / NP;
        P.d_img = dc / P.cells_img; P.d_row = dc % P.cells_img / P.IW; P.d_col = dc % P.cells_img % P.IW;
        P.d_bytes = ((P.d_img * s.H + P.d_row) * s.W + P.d_col) * P.pix_bytes;
        P.row_bytes = (s.W - P.IW) * P.pix_bytes;
        P.img_bytes = (s.H - P.IH) * s.W * P.pix_bytes;
        P.d_co = 256 / fpitch; P.d_piece = 256 % fpitch;
        P.by_tiles_y = make_fastdiv(tiles_y);
        P.by_cells_img = make_fastdiv(P.cells_img);
        P.by_IW = make_fastdiv(P.IW);
        P.by_thwo = make_fastdiv(TH * s.Wo);
        P.by_Wo = make_fastdiv(s.Wo);
        P.by_fpitch = make_fastdiv(fpitch);
        P.by_fp2 = make_fastdiv(fp2);
    };
    for (int mode = 0; mode < 4; ++mode) {
        const int CB = (mode & 1) ? 1 : 2;
        const bool fstream = mode >= 2;
        if (CB == 2 && s.C_out <= 32) continue;
        for (int PB = 1; PB <= 2; ++PB)
            for (int NP = 8; NP >= 2; NP >>= 1) {
                for (int NI = 2; NI <= s.N && (int64_t)NI * HoWo <= 128 * PB; ++NI) consider(CB, fstream, PB, NP, NI, 1);
                for (int tiles_y = 1; tiles_y <= s.Ho; ++tiles_y) consider(CB, fstream, PB, NP, 1, tiles_y);
            }
    }
    if (!best.ok) return best;
    LdsParams& P = best.P;
    P.stages = (size_t)P.win_off + 3 * (size_t)P.stage_bytes + 512 <= kLdsAll ? 3 : 2;
    P.rq_off = P.win_off + P.stages * P.stage_bytes;
    best.lds = (size_t)P.rq_off + 512;
    return best;
}

// (the search walks a few thousand candidates: more host time than a small layer runs for)
LdsPlan plan_lds(const Conv2dShape& s, int ek, const void* x, const void* w, const void* y)
{
    thread_local PlanCache<LdsPlan> cache[kFormats];
    return cache[ek].get(s, PlanCache<LdsPlan>::low_bits(x, w, y), [&] { return search_plan(s, ek, x, w, y); });
}

template <int EK, int CB, int PB, int KSC, bool FS, bool ONE>
hipError_t launch_one(const void* x, const void* w, void* y, const LdsPlan& a, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_nhwc_lds_kernel<EK, CB, PB, KSC, FS, ONE>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsAll);
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel(EK == kElemF32   ? "mfma_f32_nhwc_lds_kernel"
                                : EK == kElemF16 ? "mfma_f16_nhwc_lds_kernel"
                                : EK == kFmtS8   ? "mfma_s8_nhwc_lds_kernel"
                                : EK == kFmtS8Q  ? "mfma_s8q_nhwc_lds_kernel"
                                                 : "mfma_bf16_nhwc_lds_kernel",
                                CB + 10 * a.P.fstream, PB, a.P.NI, a.P.TH),
                    (mfma_nhwc_lds_kernel<EK, CB, PB, KSC, FS, ONE>), dim3(a.gx, a.gy), dim3(512), a.lds, st,
                    static_cast<const unsigned char*>(x), static_cast<const unsigned char*>(w), static_cast<unsigned char*>(y), a.P);
    return hipGetLastError();
}

template <int EK, int CB, int PB, int KSC, bool FS>
hipError_t launch_lds(const void* x, const void* w, void* y, const LdsPlan& a, hipStream_t st)
{
    return a.P.R * a.P.S == 1 ? launch_one<EK, CB, PB, KSC, FS, true>(x, w, y, a, st) : launch_one<EK, CB, PB, KSC, FS, false>(x, w, y, a, st);
}

}  // namespace

bool mfma_nhwc_lds_supported(const void* x, const void* w, const void* y, const Conv2dShape& s, int ek)
{
    return ek >= 0 && ek <= 2 && plan_lds(s, ek, x, w, y).ok;
}

bool mfma_s8_nhwc_lds_supported(const int8_t* x, const int8_t* w, const void* y, bool requant, const Conv2dShape& s)
{
    return s.dil == 1 && plan_lds(s, requant ? kFmtS8Q : kFmtS8, x, w, y).ok;
}

int mfma_nhwc_lds_stages(const void* x, const void* w, const void* y, const Conv2dShape& s, int fmt, int* tiles)
{
    const LdsPlan a = plan_lds(s, fmt, x, w, y);
    if (!a.ok) return 0;
    *tiles = (int)((a.tiles + a.gx - 1) / a.gx);
    return a.P.stages;
}

// fmt: Elem, kFmtS8 or kFmtS8Q
static hipError_t launch_any(const void* x, const void* w, void* y, const Conv2dShape& s, int fmt, const Epilogue& ep, const Requant& rq,
                             hipStream_t st)
{
    LdsPlan a = plan_lds(s, fmt, x, w, y);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
    a.P.rq = rq;
#define SW_K(CBC, PBC, KSC, FSC)                                                                    \
    switch (fmt) {                                                                                  \
    case kElemF32: return launch_lds<kElemF32, CBC, PBC, KSC, FSC>(x, w, y, a, st);                 \
    case kElemBF16: return launch_lds<kElemBF16, CBC, PBC, KSC, FSC>(x, w, y, a, st);               \
    case kElemF16: return launch_lds<kElemF16, CBC, PBC, KSC, FSC>(x, w, y, a, st);                 \
    case kFmtS8: return launch_lds<kFmtS8, CBC, PBC, KSC, FSC>(x, w, y, a, st);                     \
    default: return launch_lds<kFmtS8Q, CBC, PBC, KSC, FSC>(x, w, y, a, st);                        \
    }
#define SW_F(CBC, PBC, KSC) \
    { if (a.P.fstream) { SW_K(CBC, PBC, KSC, true) } else { SW_K(CBC, PBC, KSC, false) } }
#define SW_L(CBC, PBC)                        \
    if (a.CB == CBC && a.PB == PBC) {         \
        if (a.P.NP == 8) SW_F(CBC, PBC, 4)    \
        if (a.P.NP == 4) SW_F(CBC, PBC, 2)    \
        SW_F(CBC, PBC, 1)                     \
    }
    SW_L(2, 2); SW_L(2, 1); SW_L(1, 2); SW_L(1, 1);
#undef SW_K
#undef SW_F
#undef SW_L
    return hipErrorInvalidValue;
}

hipError_t launch_mfma_nhwc_lds(const void* x, const void* w, void* y, const Conv2dShape& s, int ek, const Epilogue& ep, hipStream_t st)
{
    if (ek < 0 || ek > 2) return hipErrorInvalidValue;
    return launch_any(x, w, y, s, ek, ep, Requant{nullptr, nullptr, 0}, st);
}

hipError_t launch_mfma_s8_nhwc_lds(const int8_t* x, const int8_t* w, void* y, const Requant* rq, const Conv2dShape& s, hipStream_t st)
{
    return launch_any(x, w, y, s, rq ? kFmtS8Q : kFmtS8, Epilogue{nullptr, 0}, rq ? *rq : Requant{nullptr, nullptr, 0}, st);
}

}  // namespace swconv
