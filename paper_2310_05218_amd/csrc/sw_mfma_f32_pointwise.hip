// Pointwise (1 x 1, stride 1, no padding) convolution on the matrix cores (paper, section 1.2: the pointwise stage
// of depthwise-separable convolutions; section 3: sliding sums as small matrix products).
//
//     y[n][co][p] = sum over ci of w[co][ci] * x[n][ci][p]          p = a pixel of the H x W plane
//
// With one tap there is no window: per image the sum is a plain matrix product whose B operand (channels x pixels) is
// the input tensor as it lies in memory.  The kernel therefore stages nothing of the input.  A wavefront owns 32 * QB
// consecutive pixels (counted through all images: a plane's pixel count is a multiple of QB, so the QB pixels of a lane
// never straddle two images; odd planes: see the loose form of the kernel on split operands) and CB blocks of 32 output channels.  Lane (lj, kk) of the 32 x 2 lane grid loads, for
// channel c, the QB consecutive pixels QB * lj .. QB * lj + QB - 1 with ONE load of 4 * QB bytes; element q of that
// load is its B operand for pixel block q, where block q is the pixels {QB * n + q}.  The matrix instruction does not
// care which pixel a column stands for, and on the way out the same permutation makes a lane's QB results for an
// output channel contiguous again: one 4 * QB byte store.
//
// The K index is permuted likewise: a group of eight channels is channel 4 kk + j for step j = 0..3, so the A operands
// of a lane for the four steps are four consecutive floats of a filter row, one 16-byte LDS read.  The filters of the
// workgroup's CB * 32 output channels (all of C_in) are copied to LDS once, before the first tile; after that the four
// wavefronts of a workgroup never synchronise again.  Per group of eight channels a wavefront issues 4 global loads
// and CB LDS reads for 4 * CB * QB matrix instructions (2048 cycles at CB * QB = 8); the loads run two groups ahead in
// a ring of three register sets, across tile boundaries: the next tile's first groups are requested while the current
// tile's last products run and its results are stored.
//
// Measured on 32 x 256 x 56 x 56 -> 64 (784 tiles of 128 pixels, one per wavefront): filters in LDS 3.5 us after the
// start, 33.8 us in the loop (65536 cycles of matrix instructions at the 1.94 GHz the chip holds under them: the loop
// runs at the rate of the matrix pipe), 3.8 us of stores; 46 us per launch, where the window kernels take 71 (and the kernel
// on split operands below, which has that layer since, 32.8).
#include <algorithm>

#include "sw_f32_split.h"
#include "swconv_internal.h"

namespace swconv {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr size_t kPwLdsMax = 150 * 1024;
constexpr size_t kPwLdsSplit = 156 * 1024;    // of split filters
constexpr int kRing = 3;      // register sets of B operands (measured: 4 and 6 are no faster)

struct PwParams {
    int C_in, C_out, HW;
    int total_px;     // N * H * W
    int tiles;        // of 32 * QB pixels
    int plane_groups; // (loose) groups of QB pixels of a plane; total_px counts groups then
    int wpitch;       // floats between filter rows in LDS
    FastDiv by_c4;    // 16-byte groups per filter row
    FastDiv by_oct;   // (split) groups of eight channels, rounded up to whole steps
    Epilogue ep;
};

template <int CB, int QB, int NB>
__global__ __launch_bounds__(256, 2) void mfma_f32_pointwise_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                                    float* __restrict__ y, const PwParams P)
{
    typedef float bvec __attribute__((ext_vector_type(QB)));
    extern __shared__ __attribute__((aligned(16))) float wl[];     // [CB * 32][wpitch]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lj = lane & 31, kk = lane >> 5;
    const int co0 = blockIdx.y * (CB * 32);
    const int HW = P.HW;

    const int T = P.C_in >> 3;                               // groups of eight channels
    const int nwaves = (int)gridDim.x * 4;
    int tile = (int)blockIdx.x * 4 + wave;

    // the lane's QB pixels of a tile (a lane beyond the last pixel computes on pixel 0 and stores nothing)
    struct Place {
        bool live;
        int n, pix;
    };
    auto place = [&](int tl) __attribute__((always_inline)) {
        const int pg = tl * (32 * QB) + QB * lj;
        Place p;
        p.live = tl < P.tiles && pg < P.total_px;
        const int pgc = p.live ? pg : 0;
        p.n = pgc / HW;
        p.pix = pgc - p.n * HW;
        return p;
    };
    auto x_of = [&](const Place& p) __attribute__((always_inline)) {
        return x + ((int64_t)p.n * P.C_in + 4 * kk) * HW + p.pix;      // channel 4 kk of group 0
    };

    bvec b[NB][4];
    // group g of the tile whose lane pointer is src0, into register set `buf`
    auto fetch = [&](int buf, const float* src0, int g) __attribute__((always_inline)) {
        const int gc = g < T ? g : T - 1;
        const float* src = src0 + (int64_t)(8 * gc) * HW;
#pragma unroll
        for (int j = 0; j < 4; ++j) b[buf][j] = *reinterpret_cast<const bvec*>(src + j * HW);
    };

    // the first tile's first three groups are on their way while the filters are copied
    Place cur = place(tile);
    const float* xp = x_of(cur);
#pragma unroll
    for (int i = 0; i < NB; ++i) fetch(i, xp, i);

    // filters: rows co0 .. co0 + CB * 32 - 1 (zero beyond C_out), 16 bytes at a time, eight loads in flight per thread
    {
        const int c4 = P.C_in >> 2, total = CB * 32 * c4;
#pragma unroll 1
        for (int i0 = tid; i0 < total; i0 += 8 * 256) {
            floatx4 v[8];
            int at[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int i = i0 + 256 * u, ic = i < total ? i : total - 1;
                const int row = fast_div(ic, P.by_c4), g = ic - row * c4;
                at[u] = i < total ? row * P.wpitch + 4 * g : -1;
                const int rc = co0 + row < P.C_out ? co0 + row : P.C_out - 1;
                v[u] = *reinterpret_cast<const floatx4*>(w + (int64_t)rc * P.C_in + 4 * g);
                if (co0 + row >= P.C_out) v[u] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (at[u] >= 0) *reinterpret_cast<floatx4*>(wl + at[u]) = v[u];
        }
    }
    __syncthreads();

    const float* arow = wl + lj * P.wpitch + 4 * kk;         // + cb * 32 * wpitch + 8 t
    const int T3 = T - T % NB;          // groups taken by whole trips of the main loop
#pragma unroll 1
    for (; tile < P.tiles; tile += nwaves) {
        // the wavefront's next tile: its first groups are requested while this one's last products run and its
        // results leave, so the register sets are full again when the next turn starts
        const Place nxt = place(tile + nwaves);
        const float* xq = x_of(nxt);

        floatx16 acc[CB][QB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[cb][q][v] = 0.f;

        auto read_a = [&](floatx4 (&a)[CB], int t) __attribute__((always_inline)) {
            const int tc = t < T ? t : T - 1;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) a[cb] = *reinterpret_cast<const floatx4*>(arow + cb * 32 * P.wpitch + 8 * tc);
        };
        auto multiply = [&](const floatx4 (&a)[CB], int buf) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int q = 0; q < QB; ++q)
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
                        acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[cb][j], b[buf][j][q], acc[cb][q], 0, 0, 0);
        };
        // group t of this tile, or, past its last group, group `buf` of the next tile (when the group count is a
        // multiple of NB that is exactly what set `buf` has to hold next; otherwise the groups left over after the
        // loop still need the first sets, and the next tile is requested behind them)
        auto fetch_on = [&](int buf, int t) __attribute__((always_inline)) {
            if (T3 == T && t >= T) fetch(buf, xq, buf);
            else fetch(buf, xp, t);
        };

        floatx4 a[2][CB];
        read_a(a[0], 0);
        // NB groups per trip, so that the register sets keep their names
#pragma unroll 1
        for (int t = 0; t < T3; t += NB) {
            // (the fences keep each group's loads where they are written: right behind the products that freed their
            // registers, NB - 1 groups ahead of their use)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                read_a(a[(i + 1) & 1], t + i + 1);
                multiply(a[i & 1], i);
                __builtin_amdgcn_sched_barrier(0);
                fetch_on(i, t + NB + i);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (NB & 1) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) a[0][cb] = a[1][cb];
            }
        }
        if (T3 < T) {
#pragma unroll
            for (int i = 0; i < NB - 1; ++i) {
                if (T3 + i < T) {
                    read_a(a[(i + 1) & 1], T3 + i + 1);
                    multiply(a[i & 1], i);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NB; ++i) fetch(i, xq, i);
            __builtin_amdgcn_sched_barrier(0);
        }

        // register v of a lane is output channel 8 (v / 4) + 4 kk + v % 4 of the block, pixels QB lj .. QB lj + QB - 1
        if (cur.live) {
            // (the store addresses are computed here, per tile, not kept in registers the products need: the empty
            // statement hides from the compiler that they are the same for every tile)
            int pix_out = cur.pix, kk_out = kk;
            asm volatile("" : "+v"(pix_out), "+v"(kk_out));
            float* yp = y + (int64_t)cur.n * P.C_out * HW + pix_out;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int co = co0 + cb * 32 + 8 * (v >> 2) + 4 * kk_out + (v & 3);
                    if (co < P.C_out) {
                        bvec o;
#pragma unroll
                        for (int q = 0; q < QB; ++q) o[q] = apply_epilogue(acc[cb][q][v], co, P.ep);
                        *reinterpret_cast<bvec*>(yp + (int64_t)co * HW) = o;
                    }
                }
        }
        cur = nxt;
        xp = xq;
    }
}

// The same walk on the bf16 matrix instructions, each fp32 operand as a sum of three bf16 values (sw_f32_split.h: six products
// of K = 16 take 0.375 of the fp32 instruction's time).  A K step is 16 channels, 8 kk + j for element j of lane half kk: a lane
// splits the eight values it loaded for one of its pixels, between the matrix instructions of the pixel before.  The filters
// (zeros up to the next 16 channels) are split into LDS once, before the first tile: [step][h, m, l][lane half][output channel]
// of 16 bytes.  Block and pixel counts are chosen as for the kernel above.
// Measured (us per launch, replayed graphs of ten on one set of buffers, fp32 matrix instructions -> split): 32 x 256 x 56 x 56 -> 64
// 45.7 -> 32.8, 64 -> 256 51.6 -> 44.8, 256 -> 256 at 28 x 28 42.2 -> 30.7, 512 -> 512 at 14 x 14 40.5 -> 34.1, 24 x 136 x 58 x 58 -> 16
// 25.4 -> 20.0; error against 64 bits 2.9e-7 -> 2.4e-7.  128 MB are 23 us at the rate of a large copy; the products are 13 us, one
// wavefront per SIMD.
// LOOSE: planes of any size at any 4-byte address.  A plane is taken in QB-pixel groups of its own, the last of which ends with the plane: its first
// pixels are the group before's once more, computed alike and stored twice.  Loads and stores are of 16 bytes all the same (they need no more
// than 4-byte alignment); the stores go through L2, because the nontemporal ones of the aligned form would write parts of lines.
template <int CB, int QB, int NB, bool LOOSE>
__global__ __launch_bounds__(256, CB * QB == 8 ? 1 : 2) void mfma_f32_pointwise_split_kernel(const float* __restrict__ x, const float* __restrict__ w,
                                                                                       float* __restrict__ y, const PwParams P)
{
    typedef float bvec __attribute__((ext_vector_type(QB), aligned(LOOSE ? 4 : 4 * QB)));
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    constexpr int kRow = CB * 32 + 1;                        // 16-byte units of a (step, part, lane half): odd, spreads the writes
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lj = lane & 31, kk = lane >> 5;
    const int co0 = blockIdx.y * (CB * 32);
    const int HW = P.HW;

    const int T = (P.C_in + 15) >> 4;                        // steps of sixteen channels
    const int nwaves = (int)gridDim.x * 4;
    int tile = (int)blockIdx.x * 4 + wave;

    // the lane's QB pixels of a tile (a lane beyond the last pixel computes on pixel 0 and stores nothing)
    struct Place {
        bool live;
        int n, pix;
    };
    auto place = [&](int tl) __attribute__((always_inline)) {
        Place p;
        if constexpr (LOOSE) {
            const int g = tl * 32 + lj;
            p.live = tl < P.tiles && g < P.total_px;            // (groups)
            const int gc = p.live ? g : 0;
            p.n = gc / P.plane_groups;
            p.pix = min(QB * (gc - p.n * P.plane_groups), HW - QB);
            return p;
        }
        const int pg = tl * (32 * QB) + QB * lj;
        p.live = tl < P.tiles && pg < P.total_px;
        const int pgc = p.live ? pg : 0;
        p.n = pgc / HW;
        p.pix = pgc - p.n * HW;
        return p;
    };
    auto x_of = [&](const Place& p) __attribute__((always_inline)) { return x + (int64_t)p.n * P.C_in * HW + p.pix; };

    bvec b[NB][8];
    // step g of the tile whose lane pointer is src0, into register set `buf`; a lane half without channels in the last step
    // loads the other half's (its filters are zeros)
    auto fetch = [&](int buf, const float* src0, int g) __attribute__((always_inline)) {
        const int gc = g < T ? g : T - 1;
        const int c = 16 * gc + 8 * kk;
        const float* src = src0 + (int64_t)(c < P.C_in ? c : 16 * gc) * HW;
#pragma unroll
        for (int j = 0; j < 8; ++j) b[buf][j] = *reinterpret_cast<const bvec*>(src + (int64_t)j * HW);
    };

    // the first tile's first steps are on their way while the filters are brought into LDS
    Place cur = place(tile);
    const float* xp = x_of(cur);
#pragma unroll
    for (int i = 0; i < NB; ++i) fetch(i, xp, i);

    // filters: rows co0 .. co0 + CB * 32 - 1 (zeros beyond C_out and C_in), eight channels at a time, two in flight per thread
    {
        const int octs = 2 * T, total = CB * 32 * octs;
#pragma unroll 1
        for (int i0 = tid; i0 < total; i0 += 2 * 256) {
            floatx4 v[2][2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int i = i0 + 256 * u;
                const int row = fast_div(i, P.by_oct), o = i - row * octs;
                const bool in = i < total && co0 + row < P.C_out && 8 * o < P.C_in;
                const floatx4* src = reinterpret_cast<const floatx4*>(w + (in ? (int64_t)(co0 + row) * P.C_in + 8 * o : 0));
                v[u][0] = src[0];
                v[u][1] = src[1];
                if (!in) v[u][0] = v[u][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int i = i0 + 256 * u;
                const int row = fast_div(i, P.by_oct), o = i - row * octs;
                if (i >= total) break;
                const float f[8] = {v[u][0][0], v[u][0][1], v[u][0][2], v[u][0][3], v[u][1][0], v[u][1][1], v[u][1][2], v[u][1][3]};
                const Split8 s = split_f32(f);
                bf16x8* d = reinterpret_cast<bf16x8*>(smem) + ((o >> 1) * 6 + (o & 1)) * kRow + row;
                d[0] = s.h;
                d[2 * kRow] = s.m;
                d[4 * kRow] = s.l;
            }
        }
    }
    __syncthreads();

    const int T3 = T - T % NB;          // steps taken by whole trips of the main loop
#pragma unroll 1
    for (; tile < P.tiles; tile += nwaves) {
        // the wavefront's next tile: its first steps are requested while this one's last products run and its
        // results leave, so the register sets are full again when the next turn starts
        const Place nxt = place(tile + nwaves);
        const float* xq = x_of(nxt);

        splitx16 acc[CB][QB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < QB; ++q)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[cb][q][v] = 0.f;

        auto split_pixel = [&](int buf, int q) __attribute__((always_inline)) {
            const float v[8] = {b[buf][0][q], b[buf][1][q], b[buf][2][q], b[buf][3][q], b[buf][4][q], b[buf][5][q], b[buf][6][q], b[buf][7][q]};
            return split_f32(v);
        };
        auto multiply = [&](int buf, int t) __attribute__((always_inline)) {
            Split8 a[CB], sb[2];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
                const bf16x8* s = reinterpret_cast<const bf16x8*>(smem) + (t * 6 + kk) * kRow + 32 * cb + lj;
                a[cb].h = s[0];
                a[cb].m = s[2 * kRow];
                a[cb].l = s[4 * kRow];
            }
            sb[0] = split_pixel(buf, 0);
#pragma unroll
            for (int q = 0; q < QB; ++q) {
                if (q + 1 < QB) sb[(q + 1) & 1] = split_pixel(buf, q + 1);
                const Split8& c = sb[q & 1];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cb].l, c.h, acc[cb][q], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cb].h, c.l, acc[cb][q], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cb].m, c.m, acc[cb][q], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cb].m, c.h, acc[cb][q], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cb].h, c.m, acc[cb][q], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) acc[cb][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cb].h, c.h, acc[cb][q], 0, 0, 0);
            }
            // the splitting of pixel q + 1 between the matrix instructions of pixel q
#pragma unroll
            for (int i = 0; i < 6 * CB * QB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, CB == 2 ? 5 : 10, 0);
            }
        };
        // step t of this tile, or, past its last one, step `buf` of the next tile (when the step count is a multiple of NB
        // that is exactly what set `buf` has to hold next; otherwise the steps left over after the loop still need the
        // first sets, and the next tile is requested behind them)
        auto fetch_on = [&](int buf, int t) __attribute__((always_inline)) {
            if (T3 == T && t >= T) fetch(buf, xq, buf);
            else fetch(buf, xp, t);
        };

        // NB steps per trip, so that the register sets keep their names
#pragma unroll 1
        for (int t = 0; t < T3; t += NB) {
            // (the fences keep each step's loads where they are written: right behind the products that freed their
            // registers, NB - 1 steps ahead of their use)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                multiply(i, t + i);
                __builtin_amdgcn_sched_barrier(0);
                fetch_on(i, t + NB + i);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (T3 < T) {
#pragma unroll
            for (int i = 0; i < NB - 1; ++i)
                if (T3 + i < T) multiply(i, T3 + i);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NB; ++i) fetch(i, xq, i);
            __builtin_amdgcn_sched_barrier(0);
        }

        // register v of a lane is output channel 8 (v / 4) + 4 kk + v % 4 of the block, pixels QB lj .. QB lj + QB - 1
        unsigned beyond = 0;                    // a bit per (channel block, pixel) whose accumulators hold no finite number
        if (cur.live) {
            // (the store addresses are computed here, per tile, not kept in registers the products need: the empty
            // statement hides from the compiler that they are the same for every tile)
            int pix_out = cur.pix, kk_out = kk;
            asm volatile("" : "+v"(pix_out), "+v"(kk_out));
            float* yp = y + (int64_t)cur.n * P.C_out * HW + pix_out;
            const bool whole = co0 + 32 * CB <= P.C_out;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) {
#pragma unroll
                for (int q = 0; q < QB; ++q)
                    if (split_overflow(acc[cb][q])) beyond |= 1u << (QB * cb + q);
                if constexpr (CB * QB == 8) {
                    // (accumulators in the other half of the register file: each read once)
                    float bias[16];
#pragma unroll
                    for (int v = 0; v < 16; ++v) bias[v] = 0.f;
                    if (whole && P.ep.bias) {
#pragma unroll
                        for (int v = 0; v < 16; ++v) bias[v] = P.ep.bias[co0 + cb * 32 + 8 * (v >> 2) + 4 * kk_out + (v & 3)];
                    }
#pragma unroll
                    for (int q = 0; q < QB; ++q)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[cb][q][v] = fmaf(acc[cb][q][v], kSplitUnscale, bias[v]);
                } else if (whole && P.ep.bias) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float bias = P.ep.bias[co0 + cb * 32 + 8 * (v >> 2) + 4 * kk_out + (v & 3)];
#pragma unroll
                        for (int q = 0; q < QB; ++q) acc[cb][q][v] = fmaf(acc[cb][q][v], kSplitUnscale, bias);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < QB; ++q) split_unscale(acc[cb][q]);
                }
                if (whole && P.ep.relu) {
#pragma unroll
                    for (int q = 0; q < QB; ++q)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[cb][q][v] = fmaxf(acc[cb][q][v], 0.f);
                }
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int co = co0 + cb * 32 + 8 * (v >> 2) + 4 * kk_out + (v & 3);
                    if (whole || co < P.C_out) {
                        bvec o;
#pragma unroll
                        for (int q = 0; q < QB; ++q) o[q] = whole ? acc[cb][q][v] : apply_epilogue(acc[cb][q][v], co, P.ep);
                        if constexpr (LOOSE) *reinterpret_cast<bvec*>(yp + (int64_t)co * HW) = o;
                        else __builtin_nontemporal_store(o, reinterpret_cast<bvec*>(yp + (int64_t)co * HW));
                    }
                }
            }
        }
        if (__builtin_expect(__ballot(beyond != 0) != 0, 0)) {
            int channels = P.C_in, outs = P.C_out, px = HW;         // (in vector registers: the scalar ones spilled)
            asm volatile("" : "+v"(channels), "+v"(outs), "+v"(px));
            const float* xs = x + ((int64_t)cur.n * channels + kk * (channels >> 1)) * px + cur.pix;
#pragma unroll 1
            for (int i = 0; i < CB * QB; ++i) {
                const bool mine = beyond >> i & 1;
                if (!__ballot(mine)) continue;
                const int co = co0 + 32 * (i / QB), q = i % QB;
                const splitx16 again = multiply_f32<4>(w, channels, co + lj, outs, kk, ColumnInputs{xs + q, px});
                if (mine)
                    store_outputs(again, y + ((int64_t)cur.n * outs + co + 4 * kk) * px + cur.pix + q, px, co + 4 * kk, outs, P.ep);
            }
        }
        cur = nxt;
        xp = xq;
    }
}

struct PwPlan {
    bool ok = false;
    int CB = 0, QB = 0;
    bool split = false;
    size_t lds = 0;
};

// loose: planes of any size at any 4-byte address, on split operands alone
PwPlan plan_pointwise(const Conv2dShape& s, const float* x, const float* w, const float* y, bool loose = false)
{
    PwPlan a;
    const int64_t HW = (int64_t)s.H * s.W;
    if (s.R != 1 || s.S != 1 || s.stride != 1 || s.pad != 0 || s.C_in < 8 || s.C_in % 8 != 0) return a;
    if (HW * s.N >= (1LL << 31) - (1 << 20) || HW * s.C_in >= (1LL << 31) || reinterpret_cast<uintptr_t>(w) % 16 != 0) return a;
    const auto fits = [&](int cb) { return (size_t)cb * 32 * (s.C_in + 4) * sizeof(float) <= kPwLdsMax; };
    const auto aligned = [&](int qb) {
        // A plane's last group is taken whole: of 9 pixels 12 are computed in fours, 10 in pairs.  Below 26 pixels pairs are faster, unless their
        // filters (13 steps and more of two blocks) leave a CU one workgroup.  us, fours / pairs: 72 -> 114 at 3 x 7, 2959 images 33.5 / 20.1, 40 -> 442 at
        // 3 x 3, 1648 images 28.9 / 16.6; of 308 drawn layers of 32 to 192 channels 1.12 x
        // (eleven 0.81 to 0.97), of 140 beyond 0.92 x; fewer channels stay where the direct-to-LDS kernel takes what would be fours
        if (loose) return HW >= (qb == 4 && s.C_in >= 32 && s.C_in <= 192 ? 26 : qb) && (reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y)) % 4 == 0;
        return HW % qb == 0 && reinterpret_cast<uintptr_t>(x) % (4 * qb) == 0 && reinterpret_cast<uintptr_t>(y) % (4 * qb) == 0;
    };
    const auto units = [&](int cb, int qb) {
        return ((HW * s.N + 32 * qb - 1) / (32 * qb)) * ((s.C_out + 32 * cb - 1) / (32 * cb));
    };
    // (output-channel blocks, pixel blocks) of a wavefront, in order of preference (measured: 16-byte loads and stores
    // before 8-byte ones, two channel blocks per wavefront before one); the first one that leaves every SIMD of the
    // chip a tile to work on, else the smallest that applies
    static const int kVariants[][2] = {{2, 4}, {1, 4}, {2, 2}, {1, 2}};
    for (const auto& v : kVariants) {
        if (!fits(v[0]) || !aligned(v[1])) continue;
        a.CB = v[0];
        a.QB = v[1];
        a.ok = true;
        if (units(v[0], v[1]) >= 700) break;
    }
    if (!a.ok) return a;                // (odd planes but for the loose form, filters beyond LDS)
    a.lds = (size_t)a.CB * 32 * (s.C_in + 4) * sizeof(float);
    // Split operands where their filters fit LDS, but not where the last, half empty step of 16 channels is a large part of few
    // (8 -> 32 at 256 x 256, 5 images: 15.4 us against 25.1; 72 -> 248 at 66 x 65, 7 images: 20.7 against 21.8), and from `least`
    // channels up: few channels leave little to multiply per value split and stored.  Where <2,4> has more tiles than the 1024
    // wavefronts that run at once it needs twice the rounds of the fp32 kernel, which has 2048; from two rounds of that up it makes
    // up for them.  A block of channels that is not whole is stored value by value.  us, fp32 instructions / split:
    //   fewer than 256 wavefronts: 64 -> 24, 1560 pixels 6.7 / 7.8, 152 -> 25, 858 pixels 9.8 / 10.8, 200 -> 256 at 14 x 14 12.4 / 11.9
    //   fewer than 700: 200 -> 16, 40000 pixels 12.1 / 12.6, 384 -> 384 at 14 x 14, 32 images 29.7 / 28.4
    //   <2,4>, up to 1024: 16 -> 64 at 56 x 56, 32 images 12.7 / 10.9, -> 24 9.1 / 10.5, 32 -> 24 11.1 / 11.0, 64 -> 64 19.9 / 14.9
    //   <2,4>, up to 2048: 48 to 80 channels 0.97 to 1.27 of the fp32 kernel's time, 96 channels 0.92 to 1.06
    //   <2,4>, beyond: 64 -> 256 at 56 x 56, 32 images 51.6 / 45.2, whole blocks of 32 channels 0.81 to 1.08, others 1.00 to 1.07, of
    //   48 0.73 to 1.00
    //   <2,2>: 32 channels up to 1536 wavefronts 0.86 to 1.08, 48 up to 2560 0.87 to 1.08, 64 up to 3584 0.85 to 1.11, beyond 0.95 to 1.17
    //   and 80 channels 0.80 to 1.03
    //   <1,4>: 32 -> 256 at 28 x 28, 16 images 9.8 / 8.1, 32 -> 187 at 84 x 3, 63 images 9.7 / 10.9, 48 channels 1.12
    //   <1,2>: 64 -> 61, 24534 pixels 8.2 / 9.4, 80 channels 0.99 to 1.05
    const size_t steps = (s.C_in + 15) / 16, split_lds = steps * 96 * (a.CB * 32 + 1);
    const int64_t waves = units(a.CB, a.QB);
    int least = waves < 256 ? 192 : waves < 700 ? 320 : 80;
    const bool whole = s.C_out % (32 * a.CB) == 0;
    if (waves >= 700 && a.CB * a.QB == 8) least = waves > 2048 ? (whole ? 32 : 48) : waves > 1024 ? 96 : whole ? 16 : 32;
    if (waves >= 700 && a.CB == 1 && a.QB == 4) least = waves > 2560 ? 80 : whole ? 16 : 48;
    if (waves >= 700 && a.CB == 2 && a.QB == 2) least = (int)std::min<int64_t>(80, 32 + 16 * (std::max<int64_t>(0, waves - 512) / 1024));
    a.split = split_lds <= kPwLdsSplit && (s.C_in % 16 == 0 || s.C_in >= 128) && s.C_in >= least;
    if (loose) a.split = split_lds <= kPwLdsSplit && waves >= 128 && (s.C_in >= 48 || whole || a.CB * a.QB < 8 || waves <= 1024);
    if (a.split) a.lds = split_lds;
    else if (loose) a.ok = false;
    return a;
}

template <int CB, int QB, int NB>
PwParams pw_params(const Conv2dShape& s, const Epilogue& ep, bool loose)
{
    PwParams P;
    P.C_in = s.C_in;
    P.C_out = s.C_out;
    P.HW = s.H * s.W;
    P.plane_groups = (P.HW + QB - 1) / QB;
    P.total_px = s.N * (loose ? P.plane_groups : P.HW);
    P.tiles = loose ? (P.total_px + 31) / 32 : (P.total_px + 32 * QB - 1) / (32 * QB);
    P.wpitch = s.C_in + 4;
    P.by_c4 = make_fastdiv(s.C_in / 4);
    P.by_oct = make_fastdiv(2 * ((s.C_in + 15) / 16));
    P.ep = ep;
    return P;
}

// persistent: at most two workgroups per CU (one when the filters take more than half of its LDS)
dim3 pw_grid(int tiles, int groups, size_t lds)
{
    const int per_cu = lds <= 78 * 1024 ? 2 : 1, cap = (256 * per_cu + groups - 1) / groups;
    return dim3((unsigned)std::min((tiles + 3) / 4, cap), (unsigned)groups);
}

template <int CB, int QB, int NB, bool LOOSE>
hipError_t launch_split(const float* x, const float* w, float* y, const Conv2dShape& s, const PwPlan& a, hipStream_t st, const Epilogue& ep)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_f32_pointwise_split_kernel<CB, QB, NB, LOOSE>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPwLdsSplit);
    if (attr != hipSuccess) return attr;
    const PwParams P = pw_params<CB, QB, NB>(s, ep, LOOSE);
    SW_NOTED_LAUNCH(LOOSE ? note_kernel("mfma_f32_pointwise_split_kernel", CB, QB, 1) : note_kernel("mfma_f32_pointwise_split_kernel", CB, QB),
                    (mfma_f32_pointwise_split_kernel<CB, QB, NB, LOOSE>), pw_grid(P.tiles, (s.C_out + CB * 32 - 1) / (CB * 32), a.lds), dim3(256), a.lds,
                    st, x, w, y, P);
    return hipGetLastError();
}

template <int CB, int QB, int NB>
hipError_t launch_pw(const float* x, const float* w, float* y, const Conv2dShape& s, const PwPlan& a, hipStream_t st,
                     const Epilogue& ep)
{
    if (a.split) return launch_split<CB, QB, NB, false>(x, w, y, s, a, st, ep);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_f32_pointwise_kernel<CB, QB, NB>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kPwLdsMax);
    if (attr != hipSuccess) return attr;
    const PwParams P = pw_params<CB, QB, NB>(s, ep, false);
    SW_NOTED_LAUNCH(note_kernel("mfma_f32_pointwise_kernel", CB, QB), (mfma_f32_pointwise_kernel<CB, QB, NB>),
                    pw_grid(P.tiles, (s.C_out + CB * 32 - 1) / (CB * 32), a.lds), dim3(256), a.lds, st, x, w, y, P);
    return hipGetLastError();
}

}  // namespace

bool mfma_f32_pointwise_supported(const Conv2dShape& s, const float* x, const float* w, const float* y)
{
    return plan_pointwise(s, x, w, y).ok;
}

hipError_t launch_mfma_f32_pointwise(const float* x, const float* w, float* y, const Conv2dShape& s, hipStream_t st,
                                     const Epilogue& ep)
{
    const PwPlan a = plan_pointwise(s, x, w, y);
    if (!a.ok) return hipErrorInvalidValue;
#define SW_PW(CBC, QBC) \
    if (a.CB == CBC && a.QB == QBC) return launch_pw<CBC, QBC, kRing>(x, w, y, s, a, st, ep)
    SW_PW(2, 4); SW_PW(1, 4); SW_PW(2, 2); SW_PW(1, 2);
#undef SW_PW
    return hipErrorInvalidValue;
}

// Planes that the aligned form refuses.  Against the direct-to-LDS kernel, which fetches them value by value (graph of ten, us): 152 -> 488 at 21 x 21,
// 16 images 34.7 -> 18.9; 504 -> 488 at 27 x 27, 11 images 100.6 -> 39.2; 128 -> 87 at 89 x 69, 19 images 103.7 -> 43.0; 104 -> 72 at 51 x 51, 3 images
// 14.2 -> 9.2; 56 -> 456 at 7 x 7, 23 images 12.4 -> 8.1; over 87 drawn layers 1.50.  Left to that kernel: its sums in two or four parts
// (small launches; 0.90 to 1.2, and one sum's error may be larger than that of parts), fewer than 128 units (0.95 to 1.05), more than one round of
// <2,4> with fewer than 48 channels and a block of results that is not whole (40 -> 48 at 77 x 77, 23 images 26.7 / 28.2), and fewer than 32
// channels in 16-byte groups, which are bound by the results (24 -> 248 at 63 x 63, 19 images 33.2 / 34.2; in 8-byte groups 24 -> 112 at 35 x 35, 12
// images 13.0 / 8.3).  Even planes stay on the aligned 8-byte form, 16-byte groups are 0.81 to 1.45 of it.
bool mfma_f32_pointwise_loose_supported(const Conv2dShape& s, const float* x, const float* w, const float* y)
{
    const PwPlan a = plan_pointwise(s, x, w, y, true);
    return a.ok && (s.C_in >= 32 || (s.C_in >= 16 && a.QB == 2)) && mfma_f32_dma_parts(s, x, w) <= 1;
}

hipError_t launch_mfma_f32_pointwise_loose(const float* x, const float* w, float* y, const Conv2dShape& s, hipStream_t st, const Epilogue& ep)
{
    const PwPlan a = plan_pointwise(s, x, w, y, true);
    if (!a.ok) return hipErrorInvalidValue;
    if (a.QB == 4) return a.CB == 2 ? launch_split<2, 4, kRing, true>(x, w, y, s, a, st, ep) : launch_split<1, 4, kRing, true>(x, w, y, s, a, st, ep);
    return a.CB == 2 ? launch_split<2, 2, kRing, true>(x, w, y, s, a, st, ep) : launch_split<1, 2, kRing, true>(x, w, y, s, a, st, ep);
}

}  // namespace swconv
