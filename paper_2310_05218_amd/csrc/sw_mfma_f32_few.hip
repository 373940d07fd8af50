// The multi-channel fp32 sliding sum of launches that have few tiles (one image, a late stage of a network, 5 x 5 and larger filters):
// the products of an output are split over the wavefronts of a workgroup instead of being walked through in chunks by all of them.
//
//   x [N, C_in, H, W]     w [C_out, C_in, R, S]     y [N, C_out, H_out, W_out]     fp32, any extent, stride, padding and dilation
//
// A wavefront has one tile of 16 output channels x 16 output pixels on v_mfma_f32_16x16x4_f32: the smallest tile there is gives
// the most workgroups (one image of 256 -> 256 at 14 x 14: 224).  Eight (four) wavefronts are KW x CW x PW: KW share the products of a
// tile, CW x PW have tiles of their own and share the filters' lines and the window.
//
//   window   the input cells of a workgroup's pixels, all channels of them where LDS has room (else periods of 32 channels at a time),
//            by direct-to-LDS loads, all in flight at once; padding as zeros (offsets beyond the buffer).
//   filters  straight from global memory to the registers of the operand, in the order of memory: a run of 32 products of 16 channels
//            is two 16-byte loads a lane, one line a channel; run u belongs to wavefront u mod KW, RING runs are under way.
//   cells    a product's cell (channel, tap) in the window follows from its place in the filter: a table in LDS of the 32 x taps
//            products after which the order repeats, read a run ahead.
//
// No operand is split or converted: infinities and NaN come out as fp32 arithmetic has them.  A sum is cut into KW x 12 chains of
// roundings that meet in fp32 pairs and, over the wavefronts, in fp64: 1.05e-7 of the result (2-norm) where the split operands of
// mfma_f32_split_kernel have 1.5e-7 (2304 products).
//
// Measured (us per launch, replayed graphs of ten; the kernel of before -> this one): one image of 256 -> 256 at 14 x 14 3x3 18.0 -> 10.2,
// of 512 -> 512 at 7 x 7 29.7 -> 15.7, 2 x 160 -> 40 at 11 x 11 13.4 -> 8.1, 1 x 1 over 5 x 152 -> 160 at 25 x 25 18.2 -> 10.1; 5 x 5: one
// image of 264 -> 104 at 9 x 9 658 -> 18, 8 x 176 -> 80 at 14 x 14 448 -> 37, 11 x 40 -> 64 at 39 x 39 110 -> 49.
// What bounds it (the first of these, time stamps in cycles of 19.3 k): 4.5 k until the window's loads have left (kernel arguments and tile
// coordinates 2 k; direct-to-LDS loads come in at 12 bytes a cycle and CU by words, 20 by 16-byte pieces, which need a wider window and gained
// nothing), 2.5 k first filters, the table and the wait for the window, 7 k the nine runs of two wavefronts a SIMD, 2.5 k the meeting of the sums.  An
// fp32 matrix instruction holds up the vector and LDS instructions of its SIMD: with those between them a run took 950 cycles where
// the eight matrix instructions take 290 alone and the rest 350, so they stand in one block in front.  That, uniform loop counts and no
// reads in branches: 1.07 x over 31 drawn layers (1.00 to 1.14), this one 11.1 -> 10.2 us, 10 x 80 -> 192 at 19 x 19 5 x 5 47.3 -> 41.5.
// Not where eight wavefronts run two workgroups a CU over a multiple of 32 products in 585 to 768 workgroups: of 159 such layers of 4 x 8 to 8 x 8 filters
// a third take 1.1 to 1.3 times as long as before (15 -> 167 at 71 x 22 8 x 8 stride 2, 32 images 49.4 / 62.2 us), the others 0.9 to 1.05 times.  Their wavefronts live as long
// as before, but end together, two workgroups a CU, and the last ones run alone; the order of the first ones (`stagger`) mends some.  Neither four runs of
// filters under way, with one workgroup a CU or two, nor three made up for it.
// Tried and not kept: sixteen wavefronts (12.8), loads by wavefronts of their own in four chunks with a barrier each (11.3 to 16.1), the window
// through registers by 16-byte loads (11.0, and 1 us more for the smallest layers), taps instead of runs (filters at 36-byte strides: 11.8),
// the outputs' places computed before the products (10.7).
#include <algorithm>
#include <cmath>

#include "swconv_internal.h"

namespace swconv {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef int intx4 __attribute__((ext_vector_type(4)));

#define SW_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr unsigned kBeyond = 0x80000000u;       // a byte offset no tensor of less than 2 GiB reaches

constexpr int kLds = 160 * 1024 - 256;
constexpr int kPeriod = 32;                     // channels after which the order of the products repeats in whole runs

struct FewParams {
    Epilogue ep;
    int N, C_in, C_out, H, W, Ho, Wo, stride, pad;
    int K, T, S, dil;               // products of an output, taps, filter columns
    int KW, CW, PW, lKW, lCW;       // wavefronts that share a tile's products; tiles of 16 channels; tiles of 16 pixels
    int KWq, KWr;                   // KW runs in whole periods of T and the rest
    int stagger;                    // the first of two workgroups of a CU comes first
    int TH, TW, IW, cells;          // rows and columns of a pixel tile, columns and cells of its window
    int pitch, pieces, group;       // words from a channel's window to the next's; loads per channel, or channels per load
    int CC, chunks;                 // channels in LDS at a time
    int tab_bytes;
    int co_tiles, tiles_x, tiles_y;
    unsigned x_bytes, w_bytes;
    FastDiv by_co, by_tx, by_ty, by_TW, by_IW, by_T, by_S, by_pitch;
};

// s_waitcnt vmcnt(n) alone
template <int n>
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(n) : "memory"); }

// barrier without the fence of __syncthreads (which would wait for the loads in flight)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// MIN: wavefronts that run at once on a SIMD at least; RING: runs of filters under way
template <int WAVES, int MIN, int RING>
__global__ __launch_bounds__(64 * WAVES, MIN) void mfma_f32_few_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                                                      float* __restrict__ y, const FewParams P)
{
    // Two workgroups of a CU that began together end together, and the third then runs alone: the first comes first where there are three turns of half a
    // launch's (513 to 768 workgroups; us, 28 -> 142 at 98 x 38 4 x 8 dilation 3, 6 images 60.0 -> 47.9; 159 layers 1.01 in the median, 0.93 to 1.25)
    if constexpr (WAVES == 8 && MIN == 4) {
        if (P.stagger && (blockIdx.x >> 8 & 1) == 0) __builtin_amdgcn_s_setprio(1);
    }
    constexpr int NA = 12;                              // accumulators: short chains of roundings
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    int* tab = reinterpret_cast<int*>(smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lj = lane & 15, g = lane >> 4;
    const int kw = wave & (P.KW - 1), tile = wave >> P.lKW;
    const int cw = tile & (P.CW - 1), pw = tile >> P.lCW;

    const int b = blockIdx.x;
    const int pt = fast_div(b, P.by_co), cob = b - pt * P.co_tiles;
    const int pty = fast_div(pt, P.by_tx), tx = pt - pty * P.tiles_x;
    const int n = fast_div(pty, P.by_ty), ty = pty - n * P.tiles_y;
    const int row0 = ty * P.TH, col0 = tx * P.TW, co0 = 16 * P.CW * cob;
    const int HW = P.H * P.W;

    // ---- window: the cells of `group` channels a load, or 64 cells of one channel
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, P.x_bytes, 0x00020000);
    auto stage = [&](int c0) __attribute__((always_inline)) {
        const int here = min(P.CC, P.C_in - c0);
        for (int pc = 0; pc < P.pieces; ++pc) {
            int q = 64 * pc + lane, ch = 0;
            if (P.group > 1) { ch = fast_div(lane, P.by_pitch); q = lane - ch * P.pitch; }
            const int e = fast_div(q, P.by_IW), f = q - e * P.IW;
            const int gr = row0 * P.stride - P.pad + e, gc = col0 * P.stride - P.pad + f;
            const bool in = gr >= 0 && gr < P.H && gc >= 0 && gc < P.W;
            const int step = WAVES * P.group;
            unsigned off = in ? (unsigned)(((n * P.C_in + c0 + wave * P.group + ch) * HW + gr * P.W + gc) * 4) : kBeyond;
            const unsigned inc = in ? (unsigned)(step * HW * 4) : 0;
            if (q < P.cells && ch < P.group) {
                unsigned char* d = smem + P.tab_bytes + 4 * wave * P.group * P.pitch + 256 * pc;
                for (int ci = wave * P.group; ci < here; ci += step) {
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, SW_LDS_PTR(d), 4, off, 0, 0, 0);
                    d += 4 * step * P.pitch;
                    off += inc;
                }
            }
        }
    };
    stage(0);

    // ---- filters: runs of 32 products in the order of memory, kw, kw + KW, ...; a line of each channel's filter a run
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w), 0, P.w_bytes, 0x00020000);
    const int com = co0 + 16 * cw + lj;
    const unsigned wbase = com < P.C_out ? (unsigned)((com * P.K + 4 * g) * 4) : kBeyond;
    floatx4 a[RING][2];
    const int kc = P.CC * P.T;
    auto load = [&](floatx4 (&d)[2], int k0, int u, int runs) __attribute__((always_inline)) {
        const unsigned off = u < runs ? wbase + (unsigned)((k0 + 32 * u) * 4) : kBeyond;
        d[0] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off, 0, 0));
        d[1] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off + 64, 0, 0));
    };
    int kn = min(kc, P.K), runs = kn >> 5;
#pragma unroll
    for (int i = 0; i < RING; ++i) load(a[i], 0, kw + P.KW * i, runs);

    // ---- the cell of a product of kPeriod channels: T runs
    for (int k = tid; k < min(kPeriod * P.T, P.K); k += 64 * WAVES) {
        const int ci = fast_div(k, P.by_T), tap = k - ci * P.T;
        const int r = fast_div(tap, P.by_S), s = tap - r * P.S;
        tab[k] = 4 * (ci * P.pitch + (r * P.IW + s) * P.dil);
    }
    const int p = 16 * pw + lj;
    const int pr = fast_div(p, P.by_TW), pc = p - pr * P.TW;
    const bool live = pr < P.TH && row0 + pr < P.Ho && col0 + pc < P.Wo;
    const int px = P.tab_bytes + (live ? 4 * (pr * P.IW + pc) * P.stride : 0);
    const int period = 4 * kPeriod * P.pitch;

    floatx4 acc[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) acc[i] = floatx4{0.f, 0.f, 0.f, 0.f};

    wait_loads<2 * RING>();
    for (int c = 0;; ++c) {
        lds_barrier();
        const int k0 = c * kc;
        const int mine = __builtin_amdgcn_readfirstlane((runs - kw + P.KW - 1) >> P.lKW);        // runs of this wavefront
        struct Cells { intx4 o[2]; };
        struct Vals { float v[8]; };
        int ur = kw, base = 0;                                   // the next run: its place in the table, its channels' first cell
        while (ur >= P.T) { ur -= P.T; base += period; }
        int based = base;                                        // (of the cells that wait for it)
        // the cells of run r of this wavefront; the place moves on while there are more (and no read past the last run leaves the window)
        auto cells = [&](Cells& c, int r) __attribute__((always_inline)) {
            const int* q = tab + 32 * ur + 4 * g;
            c.o[0] = *reinterpret_cast<const intx4*>(q);
            c.o[1] = *reinterpret_cast<const intx4*>(q + 16);
            based = base;
            const bool more = r + 1 < mine;
            ur += more ? P.KWr : 0;
            base += more ? P.KWq * period : 0;
            const bool turn = ur >= P.T;
            ur -= turn ? P.T : 0;
            base += turn ? period : 0;
        };
        auto places = [&](Cells& c) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) c.o[j / 4][j & 3] += px + based;
        };
        auto vals = [&](Vals& r, const Cells& c) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) r.v[j] = *reinterpret_cast<const float*>(smem + c.o[j / 4][j & 3]);
        };
        auto multiply = [&](int i, const Vals& v) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                constexpr int extra = NA - 8;
                const int k = (i & 1) && j < extra ? 8 + j : j;
                acc[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][j / 4][j & 3], v.v[j], acc[k], 0, 0, 0);
            }
        };
        if (mine > 0) {
            // Under way beside a run's matrix instructions: the next run's values, the places in LDS of those of the run after, that one's
            // successor's from the table.  In no branch: where paths with and without reads meet, the compiler waits as if there were none.
            Cells o[2];
            Vals v[2];
            cells(o[0], 0);
            places(o[0]);
            vals(v[0], o[0]);
            cells(o[0], 1);
            places(o[0]);
            cells(o[1], 2);
            int i0 = 0;
#pragma unroll 1
            for (; i0 + RING <= mine; i0 += RING) {
#pragma unroll
                for (int i = 0; i < RING; ++i) {
                    if (i0 + i > 0) load(a[(i + RING - 1) % RING], k0, kw + P.KW * (i0 + i + RING - 1), runs);
                    vals(v[(i + 1) & 1], o[i & 1]);
                    places(o[(i + 1) & 1]);
                    cells(o[i & 1], i0 + i + 3);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(i, v[i & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int i = 0; i < RING - 1; ++i)
                if (i0 + i < mine) {
                    if (i + 1 < RING - 1) {
                        vals(v[(i + 1) & 1], o[i & 1]);
                        places(o[(i + 1) & 1]);
                        cells(o[i & 1], i0 + i + 3);
                    }
                    multiply(i, v[i & 1]);
                }
        }
        // the last products, less than a run
        if ((kn & 31) && kw == (runs & (P.KW - 1))) {
            int place = runs, from = px;
            while (place >= P.T) { place -= P.T; from += period; }
#pragma unroll 1
            for (int k = 0; k < (kn & 31); k += 4) {
                const bool in = k + g < (kn & 31);
                const float av = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(wr, in ? wbase + (unsigned)((k0 + 32 * runs + k - 3 * g) * 4) : kBeyond, 0, 0));
                const float bv = *reinterpret_cast<const float*>(smem + (from + tab[32 * place + (in ? k + g : k)]));
                acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, in ? bv : 0.f, acc[0], 0, 0, 0);
            }
        }
        if (c + 1 == P.chunks) break;
        lds_barrier();
        stage((c + 1) * P.CC);
        kn = __builtin_amdgcn_readfirstlane(min(kc, P.K - (c + 1) * kc));
        runs = kn >> 5;
#pragma unroll
        for (int i = 0; i < RING; ++i) load(a[i], (c + 1) * kc, kw + P.KW * i, runs);
        wait_loads<2 * RING>();
    }

    // ---- the parts of a tile's sums meet in LDS
#pragma unroll
    for (int i = 8; i < NA; ++i) acc[i - 8] += acc[i];
    const floatx4 sum = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
    float* red = reinterpret_cast<float*>(smem);
    lds_barrier();
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave * 256 + (4 * g + v) * 16 + lj] = sum[v];
    lds_barrier();
    for (int o = tid; o < 256 * P.CW * P.PW; o += 64 * WAVES) {
        const int ot = o >> 8, m = (o >> 4) & 15, q = 16 * (ot >> P.lCW) + (o & 15);
        const int qr = fast_div(q, P.by_TW), qc = q - qr * P.TW;
        const int co = co0 + 16 * (ot & (P.CW - 1)) + m;
        double s = 0;                                   // (in fp32 these few additions were a third of the error of a short sum)
        for (int i = 0; i < P.KW; ++i) s += (double)red[(ot * P.KW + i) * 256 + (o & 255)];
        if (co < P.C_out && qr < P.TH && row0 + qr < P.Ho && col0 + qc < P.Wo)
            y[(((int64_t)n * P.C_out + co) * P.Ho + row0 + qr) * P.Wo + col0 + qc] = apply_epilogue((float)s, co, P.ep);
    }
}

struct FewPlan {
    bool ok = false;
    int waves = 0, lds = 0;
    int64_t grid = 0;
    double est = 0;
    FewParams P;
};

FewPlan search_few(const Conv2dShape& s)
{
    FewPlan best;
    const int64_t x_bytes = (int64_t)s.N * s.C_in * s.H * s.W * 4, w_bytes = (int64_t)s.C_out * s.C_in * s.R * s.S * 4;
    // (the channels that a load takes beyond the last are read: their offsets stay below 2^31 as well)
    if (x_bytes + 256LL * s.H * s.W >= (1LL << 31) || w_bytes >= (1LL << 31)) return best;
    const int T = s.R * s.S;
    const int64_t K = (int64_t)s.C_in * T, span_r = (int64_t)(s.R - 1) * s.dil + 1, span_s = (int64_t)(s.S - 1) * s.dil + 1;
    if (span_r > 4096 || span_s > 4096) return best;
    auto consider = [&](int waves, int KW, int CW, int PW, int TW) {
        const int TH = std::min(s.Ho, 16 * PW / TW);
        const int64_t IH = (int64_t)(TH - 1) * s.stride + span_r, IW = (int64_t)(TW - 1) * s.stride + span_s;
        if (IH * IW > 4096) return;
        const int cells = (int)(IH * IW);
        // (a pitch that puts the reads of the four lane groups on different banks)
        const int pitch = cells > 32 ? cells + (48 - cells % 32) % 32 : cells > 21 ? 32 : cells > 16 ? 21 : cells > 12 ? 16 : cells;
        const int pieces = (cells + 63) / 64, group = cells <= 32 ? 64 / pitch : 1;
        const int tab_bytes = (int)std::min<int64_t>(kPeriod * T, K + 3) * 4 / 16 * 16 + 16;
        // channels in LDS at a time: all, or as many whole periods as there is room for
        const int room = (kLds - tab_bytes) / (4 * pitch) - group;
        const int CC = s.C_in <= room ? s.C_in : room / kPeriod * kPeriod;
        if (CC <= 0) return;
        const int chunks = (s.C_in + CC - 1) / CC;
        const int lds = std::max(tab_bytes + (CC + group) * pitch * 4, waves * 1024);
        const int ty = (s.Ho + TH - 1) / TH, tx = (s.Wo + TW - 1) / TW, cot = (s.C_out + 16 * CW - 1) / (16 * CW);
        const int64_t grid = (int64_t)s.N * ty * tx * cot;
        if (grid >= (1LL << 22) || grid * std::max(cot, std::max(tx, ty)) >= (1LL << 32)) return;      // (fast_div's range)
        // us, fitted to 2300 launches of 220 layers (12 splits each): the matrix instructions at 1.8 of a CU's thousand cycles a us, a
        // third more where a SIMD has one wavefront only; the loads of the window and of the filters; what a workgroup does once
        const int percu = std::min(kLds / (lds + 512), 16 / waves);
        const double rounds = std::ceil((double)grid / (256.0 * std::max(percu, 1)));
        const double turns = grid > 512 ? grid / 256.0 : std::ceil(grid / 256.0);
        const int64_t at_once = std::min<int64_t>(std::max(percu, 1), (grid + 255) / 256);
        double mul = 0;
        for (int c = 0; c < chunks; ++c) {
            const int64_t runs = ((int64_t)std::min(CC, s.C_in - c * CC) * T + 31) / 32;
            mul += (double)((runs + KW - 1) / KW) * 8 * 32 * (waves / 4) * 1e-3;
        }
        const double window = (double)((s.C_in + group - 1) / group) * pieces * 1e-2, filters = (double)CW * PW * ((K + 31) / 32) * 2e-2;
        const double est = 2.24 + turns * ((waves * at_once <= 4 ? 0.90 : 0.57) * mul + 0.83 * window + 0.81 * filters) + 3.0 * rounds * chunks;
        if (best.ok && est >= best.est) return;
        best.ok = true;
        best.est = est;
        best.waves = waves; best.lds = lds; best.grid = grid;
        FewParams& P = best.P;
        P.N = s.N; P.C_in = s.C_in; P.C_out = s.C_out; P.H = s.H; P.W = s.W; P.Ho = s.Ho; P.Wo = s.Wo;
        P.stride = s.stride; P.pad = s.pad; P.dil = s.dil;
        P.K = (int)K; P.T = T; P.S = s.S;
        P.KW = KW; P.CW = CW; P.PW = PW; P.KWq = KW / T; P.KWr = KW % T; P.lKW = __builtin_ctz(KW); P.lCW = __builtin_ctz(CW);
        P.TH = TH; P.TW = TW; P.IW = (int)IW; P.cells = cells; P.pitch = pitch; P.pieces = pieces; P.group = group;
        P.CC = CC; P.chunks = chunks; P.tab_bytes = tab_bytes;
        P.co_tiles = cot; P.tiles_x = tx; P.tiles_y = ty;
        P.x_bytes = (unsigned)x_bytes; P.w_bytes = (unsigned)w_bytes;
        P.by_co = make_fastdiv(cot); P.by_tx = make_fastdiv(tx); P.by_ty = make_fastdiv(ty); P.by_TW = make_fastdiv(TW);
        P.by_IW = make_fastdiv((int)IW); P.by_T = make_fastdiv(T); P.by_S = make_fastdiv(s.S); P.by_pitch = make_fastdiv(pitch);
    };
    for (int waves : {8, 4})
        for (int KW = waves; KW >= 1; KW /= 2)
            for (int CW = 1; CW * KW <= waves; CW *= 2) {
                const int PW = waves / KW / CW;
                // columns of a tile: equal parts of an output row, the twelve widest (TW - 1 columns or fewer from as many parts up)
                int TW = 0;
                for (int64_t nx = std::max(1, (s.Wo + 16 * PW - 1) / (16 * PW)), tried = 0; tried < 12 && TW != 1; nx = ((int64_t)s.Wo + TW - 2) / std::max(TW - 1, 1), ++tried) {
                    TW = (int)((s.Wo + nx - 1) / nx);
                    if (TW < std::min(s.Wo, 4)) break;                                      // (narrow tiles: scattered loads and stores)
                    consider(waves, KW, CW, PW, TW);
                }
            }
    return best;
}

FewPlan plan_few(const Conv2dShape& s)
{
    thread_local PlanCache<FewPlan> cache;
    return cache.get(s, 0, [&] { return search_few(s); });
}

template <int WAVES, int MIN, int RING>
hipError_t launch_one(const float* x, const float* w, float* y, const FewPlan& a, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_f32_few_kernel<WAVES, MIN, RING>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel("mfma_f32_few_kernel", WAVES, a.P.KW, a.P.PW, a.P.chunks), (mfma_f32_few_kernel<WAVES, MIN, RING>),
                    dim3((unsigned)a.grid), dim3(64 * WAVES), a.lds, st, x, w, y, a.P);
    return hipGetLastError();
}

}  // namespace

bool mfma_f32_few_supported(const Conv2dShape& s) { return plan_few(s).ok; }

double mfma_f32_few_estimate(const Conv2dShape& s) { return plan_few(s).est; }

int mfma_f32_few_columns(const Conv2dShape& s) { return plan_few(s).P.TW; }

hipError_t launch_mfma_f32_few(const float* x, const float* w, float* y, const Conv2dShape& s, hipStream_t st, const Epilogue& ep)
{
    FewPlan a = plan_few(s);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
    a.P.stagger = a.grid > 512 && a.grid <= 768;
    // four wavefronts: a fourth workgroup a CU likewise (graph of ten, us, four filters under way / two: 208 -> 16 at 31 x 31, 15 images 11.7 / 10.8, 96
    // -> 16 at 31 x 31, 27 images 9.7 / 8.8); with 768 workgroups or fewer all run at once as it is
    if (a.waves == 4)
        return a.grid > 768 && 4 * (a.lds + 512) <= 160 * 1024 ? launch_one<4, 4, 2>(x, w, y, a, st) : launch_one<4, 2, 4>(x, w, y, a, st);
    // eight wavefronts: two workgroups a CU, with half the filters under way, where there are that many and LDS has room for them
    return a.grid > 256 && 2 * (a.lds + 512) <= 160 * 1024 ? launch_one<8, 4, 2>(x, w, y, a, st) : launch_one<8, 2, 4>(x, w, y, a, st);
}

}  // namespace swconv
