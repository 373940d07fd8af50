// int8 convolution on channel-first tensors with one or nine taps (exact int32 sums, leaving as int32 or requantised to int8): a tile of
// 16 output channels x 16 PB output pixels per wavefront, operands byte-transposed once on their way to the matrix instruction.
//
//   x [N, C_in, H, W]     w [C_out, C_in, R, S]     y [N, C_out, H_out, W_out]     C_in in whole groups of 16, any stride and padding
//
// v_mfma_i32_16x16x64_i8 wants 16 consecutive channels of a pixel (of a tap) in a lane; the tensors keep them a plane (a tap count) apart.
//
//   window   [channel group of 16][cell] of 16 bytes in LDS: the input cells of a workgroup's pixels, padding as zeros.  A lane loads four
//            columns of a row of 16 channels (16 dwords) and turns them in registers: 32 v_perm for 64 bytes.  At a row's end it takes the
//            last four columns that exist: what overlaps is written twice with the same values.
//   filters  16 channels x nine taps of an output channel are 144 consecutive bytes: nine 16-byte loads a lane, 108 v_perm, the next unit's
//            loads in flight.  A single tap needs no turning.
//
// Eight wavefronts are KW x CW x PW: KW share a tile's units of 64 channels and add up through LDS, CW x PW have tiles of their own.
//
// Measured (us per launch, replayed graphs of ten; mfma_s8_any_kernel -> this one): 8 x 224 -> 80 at 14 x 53 3x3 stride 2, requantised, 87 -> 7.3;
// 2 x 352 -> 208 at 10 x 10 3x3 76 -> 6.3; 32 x 512 -> 512 at 14 x 14 3x3 137 -> 49; 16 x 112 -> 192 at 112 x 112 3x3 297 -> 130; 4 x 208 -> 64
// at 61 x 61 1x1 23 -> 5.7; 370 drawn layers 3.8 x (geometric mean).
// What bounds it: small launches the round trip, the turning and the barriers (4.1 us the smallest); large ones the turning of the
// filters, once per 16 PB pixels (450 cycles for 64 channels, nine taps, where the matrix instructions take 144 PB).
#include <algorithm>
#include <cmath>

#include "sw_s8_perm.h"
#include "swconv_internal.h"

namespace swconv {

namespace {

using s8perm::intx4;
using s8perm::u32;
using s8perm::perm;

constexpr unsigned kBeyond = 0x80000000u;       // a byte offset no tensor of less than 2 GiB reaches
constexpr int kLds = 160 * 1024 - 512;
constexpr int kThreads = 512;
constexpr int kMaxTaps = 9;

struct S8TilesParams {
    Requant rq;
    int N, C_in, C_out, H, W, Ho, Wo, stride, pad;
    int C16, units;                 // groups of 16 input channels, units of 64
    int KW, CW, lKW, lCW;           // wavefronts that share a tile's units; tiles of 16 output channels
    int TH, TW, IW, cells;          // rows and columns of a pixel tile, columns and cells of its window
    int NQ, per16, items;           // quads of window columns, (row, quad)s of a channel group, of the window
    int rq_off;
    int co_tiles, tiles_x, tiles_y;
    int off[kMaxTaps];              // bytes from a pixel's first cell to a tap's
    unsigned w_bytes;
    FastDiv by_co, by_tx, by_ty, by_TW, by_rq, by_NQ;
};

__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// T: taps (1 or 9).  PB: tiles of 16 pixels per wavefront.
template <int T, int PB, bool RQ>
__global__ __launch_bounds__(kThreads, 4) void mfma_s8_tiles_kernel(const int8_t* __restrict__ x, const int8_t* __restrict__ w, int32_t* __restrict__ y,
                                                                  int8_t* __restrict__ y8, const S8TilesParams P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
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

    // ---- window: an item is four columns of a row of 16 channels; four columns that exist, where the row's end is nearer
    const int top = row0 * P.stride - P.pad, left = col0 * P.stride - P.pad;
    const int lo = max(left, 0), hi = min(P.W, left + P.IW);
    const int8_t* const xn = x + (int64_t)n * P.C_in * HW;
    u32 raw[16];
    int dst = 0, from = 0;
    bool have = false;
    auto fetch = [&](int i) __attribute__((always_inline)) {
        const int c16 = fast_div(i, P.by_rq), rem = i - c16 * P.per16;
        const int e = fast_div(rem, P.by_NQ), q = rem - e * P.NQ;
        const int gr = top + e;
        from = max(min(lo + 4 * q, hi - 4), 0);
        have = i < P.items && gr >= 0 && gr < P.H && lo + 4 * q < hi;
        dst = 16 * (c16 * P.cells + e * P.IW + from - left);
        if (have) {
            const int8_t* p = xn + (16 * c16 * HW + gr * P.W + from);
#pragma unroll
            for (int j = 0; j < 16; ++j) __builtin_memcpy(&raw[j], p + j * HW, 4);
        }
    };
    auto put = [&]() __attribute__((always_inline)) {
        if (!have) return;
        intx4 cell[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) {                   // 4 x 4 bytes: channels 4 a ... of four pixels
            const u32 l01 = perm(raw[4 * a + 1], raw[4 * a], 0x05010400u), h01 = perm(raw[4 * a + 1], raw[4 * a], 0x07030602u);
            const u32 l23 = perm(raw[4 * a + 3], raw[4 * a + 2], 0x05010400u), h23 = perm(raw[4 * a + 3], raw[4 * a + 2], 0x07030602u);
            cell[0][a] = (int)perm(l23, l01, 0x05040100u);
            cell[1][a] = (int)perm(l23, l01, 0x07060302u);
            cell[2][a] = (int)perm(h23, h01, 0x05040100u);
            cell[3][a] = (int)perm(h23, h01, 0x07060302u);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (from + j >= lo && from + j < hi) *reinterpret_cast<intx4*>(smem + dst + 16 * j) = cell[j];
    };
    fetch(tid);

    // ---- filters: 16 channels x T taps of one output channel are T consecutive 16-byte pieces
    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(w), 0, P.w_bytes, 0x00020000);
    const int com = co0 + 16 * cw + lj;
    const unsigned wbase = com < P.C_out ? (unsigned)(com * P.C_in * T) : kBeyond;
    u32 f[4 * T];
    auto load = [&](int u) __attribute__((always_inline)) {
        const int c16 = 4 * u + g;
        const unsigned off = c16 < P.C16 ? wbase + (unsigned)(16 * T * c16) : kBeyond;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const intx4 v = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(wr, off + 16 * t, 0, 0));
#pragma unroll
            for (int j = 0; j < 4; ++j) f[4 * t + j] = (u32)v[j];
        }
    };
    load(kw);

    // ---- padding
    for (int i = tid; i < P.C16 * P.cells; i += kThreads) *reinterpret_cast<intx4*>(smem + 16 * i) = intx4{0, 0, 0, 0};
    if constexpr (RQ) {
        if (tid < 16 * P.CW) {
            const int co = co0 + tid;
            reinterpret_cast<int*>(smem + P.rq_off)[tid] = P.rq.bias != nullptr && co < P.C_out ? P.rq.bias[co] : 0;
            reinterpret_cast<float*>(smem + P.rq_off)[16 * P.CW + tid] = co < P.C_out ? P.rq.scale[co] : 0.f;
        }
    }
    lds_barrier();
    put();
    for (int i = tid + kThreads; i < P.items; i += kThreads) {
        fetch(i);
        put();
    }

    int px[PB];
#pragma unroll
    for (int q = 0; q < PB; ++q) {
        const int p = 16 * (PB * pw + q) + lj;
        const int pr = fast_div(p, P.by_TW), pc = p - pr * P.TW;
        px[q] = pr < P.TH && row0 + pr < P.Ho && col0 + pc < P.Wo ? 16 * (pr * P.IW + pc) * P.stride : 0;
    }
    intx4 acc[PB];
#pragma unroll
    for (int q = 0; q < PB; ++q) acc[q] = intx4{0, 0, 0, 0};
    lds_barrier();

#pragma unroll 1
    for (int u = kw; u < P.units; u += P.KW) {
        intx4 a[T];
        if constexpr (T == 9) {
            a[0] = s8perm::wgather_tap<0>(f); a[1] = s8perm::wgather_tap<1>(f); a[2] = s8perm::wgather_tap<2>(f);
            a[3] = s8perm::wgather_tap<3>(f); a[4] = s8perm::wgather_tap<4>(f); a[5] = s8perm::wgather_tap<5>(f);
            a[6] = s8perm::wgather_tap<6>(f); a[7] = s8perm::wgather_tap<7>(f); a[8] = s8perm::wgather_tap<8>(f);
        } else {
            a[0] = intx4{(int)f[0], (int)f[1], (int)f[2], (int)f[3]};
        }
        const int group = 16 * P.cells * min(4 * u + g, P.C16 - 1);     // (channels beyond the last have zeros for filters)
        if (u + P.KW < P.units) load(u + P.KW);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int q = 0; q < PB; ++q)
                acc[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t], *reinterpret_cast<const intx4*>(smem + (group + px[q] + P.off[t])), acc[q], 0, 0, 0);
    }

    auto store = [&](int sum, int m, int q) __attribute__((always_inline)) {
        const int qr = fast_div(q, P.by_TW), qc = q - qr * P.TW;
        const int co = co0 + m;
        if (co >= P.C_out || qr >= P.TH || row0 + qr >= P.Ho || col0 + qc >= P.Wo) return;
        const int64_t at = (((int64_t)n * P.C_out + co) * P.Ho + row0 + qr) * P.Wo + col0 + qc;
        if constexpr (RQ) {
            float r = rintf(__int2float_rn(sum + reinterpret_cast<const int*>(smem + P.rq_off)[m]) * reinterpret_cast<const float*>(smem + P.rq_off)[16 * P.CW + m]);
            r = fminf(fmaxf(r, P.rq.relu ? 0.0f : -128.0f), 127.0f);
            y8[at] = (int8_t)(int)r;
        } else {
            y[at] = sum;
        }
    };
    if (P.KW == 1) {
#pragma unroll
        for (int q = 0; q < PB; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) store(acc[q][v], 16 * cw + 4 * g + v, 16 * (PB * pw + q) + lj);
        return;
    }
    // ---- the parts of a tile's sums meet in LDS
    int* red = reinterpret_cast<int*>(smem);
    lds_barrier();
#pragma unroll
    for (int q = 0; q < PB; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[(wave * PB + q) * 256 + (4 * g + v) * 16 + lj] = acc[q][v];
    lds_barrier();
    const int tiles = 8 >> P.lKW;
    for (int o = tid; o < 256 * PB * tiles; o += kThreads) {
        const int ot = o / (256 * PB), q = (o >> 8) & (PB - 1);
        int s = 0;
        for (int i = 0; i < P.KW; ++i) s += red[((ot * P.KW + i) * PB + q) * 256 + (o & 255)];
        store(s, 16 * (ot & (P.CW - 1)) + ((o >> 4) & 15), 16 * (PB * (ot >> P.lCW) + q) + (o & 15));
    }
}

struct S8TilesPlan {
    bool ok = false;
    int PB = 0, lds = 0;
    int64_t grid = 0;
    double est = 0;
    S8TilesParams P;
};

S8TilesPlan search_s8_tiles(const Conv2dShape& s, bool requant)
{
    S8TilesPlan best;
    const int T = s.R * s.S;
    const int64_t x_bytes = (int64_t)s.N * s.C_in * s.H * s.W, w_bytes = (int64_t)s.C_out * s.C_in * T;
    if ((T != 1 && T != 9) || s.C_in % 16 != 0 || s.W < 4 || s.dil != 1 || x_bytes >= (1LL << 31) || w_bytes >= (1LL << 31)) return best;
    const int C16 = s.C_in / 16, units = (C16 + 3) / 4;
    auto consider = [&](int KW, int CW, int PB, int TW) {
        const int px = 16 * PB * (8 / KW / CW);
        if (TW > px) return;
        const int TH = std::min(s.Ho, px / TW);
        const int64_t IH = (int64_t)(TH - 1) * s.stride + s.R, IW = (int64_t)(TW - 1) * s.stride + s.S;
        if (IH * IW * s.C_in > kLds - 1024) return;
        const int cells = (int)(IH * IW), NQ = (int)(IW + 3) / 4, items = C16 * (int)IH * NQ;
        const int rq_off = std::max(C16 * cells * 16, KW > 1 ? 8 * PB * 1024 : 0), lds = rq_off + 128 * CW;
        if (lds > kLds) return;
        const int ty = (s.Ho + TH - 1) / TH, tx = (s.Wo + TW - 1) / TW, cot = (s.C_out + 16 * CW - 1) / (16 * CW);
        const int64_t grid = (int64_t)s.N * ty * tx * cot;
        if (grid >= (1LL << 22) || grid * std::max(cot, std::max(tx, ty)) >= (1LL << 32)) return;
        const int percu = std::min(kLds / (lds + 512), 2);
        const double rounds = std::ceil((double)grid / (256.0 * std::max(percu, 1)));
        const double turns = grid > 512 ? grid / 256.0 : std::ceil(grid / 256.0);
        // us, fitted to 6000 launches of 220 layers (30 splits each)
        const double mine = (double)((units + KW - 1) / KW);
        const int ob = requant ? 1 : 4;
        const double est = 3.42 + turns * (mine * (T == 9 ? 0.22 : 0.0) + mine * T * (0.35 * PB + 0.46) / 9 + 0.2 * items / kThreads + 0.35 * cells * C16 / kThreads +
                                           2.1e-3 * 16 * CW * TH * ((TW * ob + 63) / 64)) + (KW > 1 ? 0.81 : 0.43) * rounds;
        if (best.ok && est >= best.est) return;
        best.ok = true; best.est = est; best.PB = PB; best.lds = lds; best.grid = grid;
        S8TilesParams& P = best.P;
        P.N = s.N; P.C_in = s.C_in; P.C_out = s.C_out; P.H = s.H; P.W = s.W; P.Ho = s.Ho; P.Wo = s.Wo; P.stride = s.stride; P.pad = s.pad;
        P.C16 = C16; P.units = units; P.KW = KW; P.CW = CW; P.lKW = __builtin_ctz(KW); P.lCW = __builtin_ctz(CW);
        P.TH = TH; P.TW = TW; P.IW = (int)IW; P.cells = cells; P.NQ = NQ; P.items = items; P.per16 = (int)IH * NQ; P.rq_off = rq_off;
        P.co_tiles = cot; P.tiles_x = tx; P.tiles_y = ty; P.w_bytes = (unsigned)w_bytes;
        for (int t = 0; t < T; ++t) P.off[t] = 16 * ((t / s.S) * (int)IW + t % s.S);
        P.by_co = make_fastdiv(cot); P.by_tx = make_fastdiv(tx); P.by_ty = make_fastdiv(ty); P.by_TW = make_fastdiv(TW);
        P.by_rq = make_fastdiv((int)IH * NQ); P.by_NQ = make_fastdiv(NQ);
    };
    for (int KW = 8; KW >= 1; KW /= 2)
        for (int CW = 1; CW * KW <= 8; CW *= 2)
            for (int PB : {1, 2, 4}) {
                const int px = 16 * PB * (8 / KW / CW);
                // columns of a tile: equal parts of an output row, the twelve widest (TW - 1 columns or fewer from as many parts up)
                int TW = 0;
                for (int64_t nx = std::max(1, (s.Wo + px - 1) / px), tried = 0; tried < 12 && TW != 1; nx = ((int64_t)s.Wo + TW - 2) / std::max(TW - 1, 1), ++tried) {
                    TW = (int)((s.Wo + nx - 1) / nx);
                    if (TW < std::min(s.Wo, 4)) break;
                    consider(KW, CW, PB, TW);
                }
            }
    return best;
}

S8TilesPlan plan_s8_tiles(const Conv2dShape& s, bool requant)
{
    thread_local PlanCache<S8TilesPlan> cache[2];
    return cache[requant].get(s, 0, [&] { return search_s8_tiles(s, requant); });
}

template <int T, int PB, bool RQ>
hipError_t launch_one(const int8_t* x, const int8_t* w, int32_t* y, int8_t* y8, const S8TilesPlan& a, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_s8_tiles_kernel<T, PB, RQ>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel("mfma_s8_tiles_kernel", T, a.P.KW, a.P.CW, PB), (mfma_s8_tiles_kernel<T, PB, RQ>),
                    dim3((unsigned)a.grid), dim3(kThreads), a.lds, st, x, w, y, y8, a.P);
    return hipGetLastError();
}

}  // namespace

bool mfma_s8_tiles_supported(const int8_t* w, bool requant, const Conv2dShape& s) { return reinterpret_cast<uintptr_t>(w) % 4 == 0 && plan_s8_tiles(s, requant).ok; }

hipError_t launch_mfma_s8_tiles(const int8_t* x, const int8_t* w, int32_t* y, int8_t* y8, const Requant* rq, const Conv2dShape& s, hipStream_t st)
{
    S8TilesPlan a = plan_s8_tiles(s, rq != nullptr);
    if (!a.ok) return hipErrorInvalidValue;
    if (rq) a.P.rq = *rq;
#define SW_PB(TC, RQC)                                                \
    switch (a.PB) {                                                   \
    case 1: return launch_one<TC, 1, RQC>(x, w, y, y8, a, st);        \
    case 2: return launch_one<TC, 2, RQC>(x, w, y, y8, a, st);        \
    default: return launch_one<TC, 4, RQC>(x, w, y, y8, a, st);       \
    }
    if (s.R * s.S == 9) { if (rq) SW_PB(9, true) else SW_PB(9, false) }
    if (rq) SW_PB(1, true) else SW_PB(1, false)
#undef SW_PB
}

}  // namespace swconv
