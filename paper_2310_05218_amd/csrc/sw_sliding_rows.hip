// 2-D sliding window sums with one filter per plane (or none: pooling), small fixed windows, stride 1
// or 2, held entirely in registers: no LDS (paper, section 2: the "custom" kernels for small fixed
// sizes; abstract: pooling and convolution are the same sliding sum).
//
// A wavefront owns a strip of 256 input columns (one aligned 16-byte load per lane and input row: 1 KB
// per row, fully coalesced) and a band of TR output rows.  At stride 1 a lane's four outputs of a row
// sit at the same columns as its four inputs, at stride 2 its two outputs sit at half that column, so
// loads and stores are both aligned; the taps that reach across the lane boundary take `pad` values
// from the left neighbour and the rest from the right one, moved with DPP wavefront shifts
// (v_mov_b32_dpp wave_shr:1 / wave_shl:1) -- the row shift of the sliding sum.
// Vertically every input row is loaded once per band and accumulated into each output row it meets
// (choice of accumulator row).  Strips overlap by one lane on each inner side, because the edge lanes
// have no neighbour to take the halo from; at the image border the shifted-in value is the padding
// itself (zero for sums, minus infinity for the maximum, which padding must never win).
// All row loads of a band are issued before the first use, so a band costs one memory round trip.
//
// Measured (us per launch, replayed graphs of ten; before -> with loads that no branch guards): one image of 256 x 256 under 3x3
// 5.1 -> 3.75, seven of 423 x 480 under 5x5 7.6 -> 5.5, depthwise 5x5 on 14 x 184 x 18 x 84 19.1 -> 9.5, at stride 2 on 32 x 300 x 400
// 11.0 -> 5.1.  With a branch around every row's load the compiler copied the rows from register to register at each join (133 to
// 216 registers for 24 to 68 in use, three waves per SIMD or two); an address clamped into the image and a select take none.
// Bound by bytes where the planes fill the chip (3x3 pooling at stride 2 on 32 x 64 x 112 x 112: 20.3, 6.3 TB/s), by one memory round
// trip and the launch where they do not.
#include "swconv_internal.h"

#include <algorithm>
#include <cmath>

namespace swconv {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float floatx2u __attribute__((ext_vector_type(2), aligned(4)));

constexpr int kStripIn = 256;             // input columns per wavefront
constexpr int kStripFirst = 252;          // input columns whose lanes have both neighbours, first strip
constexpr int kStripStep = 248;           // distance between strip origins (lanes 1..62 of later strips)

enum RowsOp { ROWS_CONV = 0, ROWS_AVG = 1, ROWS_MAX = 2 };

// lane i receives lane i-1's value (from_left) or lane i+1's (from_right); the lane without such a
// neighbour receives FILL
template <int OP>
__device__ __forceinline__ float from_left(float v)
{
    if constexpr (OP == ROWS_MAX)
        return __int_as_float(__builtin_amdgcn_update_dpp((int)0xff800000, __float_as_int(v), 0x138, 0xF, 0xF, false));
    else
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
template <int OP>
__device__ __forceinline__ float from_right(float v)
{
    if constexpr (OP == ROWS_MAX)
        return __int_as_float(__builtin_amdgcn_update_dpp((int)0xff800000, __float_as_int(v), 0x130, 0xF, 0xF, false));
    else
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}

// A wavefront's place among strips, bands and planes, without the integer divide sequence (64-bit as they were, the four divisions took
// a third of a microsecond of a launch: 5.12 -> 4.75 us for one image of 256 x 256) where the numbers are in fast_div's range.
struct RowsPlace {
    FastDiv by_strips, by_bands, by_planes_per_x, by_filters;
    int wide;                       // a number beyond fast_div's range: the integer divide sequence
    __device__ __forceinline__ int div(int n, FastDiv f) const { return wide ? (int)((uint32_t)n / f.d) : fast_div(n, f); }
};

// PADC: padding (compile time).  ST: stride, 1 or 2.  OP: weighted sum, average or maximum.
// SEGL: lanes per work item.  64: the wavefront walks strips of a wide plane.  8, 16 or 32: planes narrower
// than 4 * SEGL columns, one (plane, band) item per group of SEGL lanes; the lanes of a group beyond the
// plane's width hold padding, which is exactly what the neighbouring group's edge lane must shift in.
// ANY: rows that begin at any 4-byte address and end inside a lane's four columns.
template <int R, int S, int PADC, int TR, int ST, int OP, int SEGL, bool ANY>
__global__ __launch_bounds__(256) void sliding_rows_kernel(const float* __restrict__ x,
                                                           const float* __restrict__ w,
                                                           float* __restrict__ y, int H, int W, int Ho, int Wo,
                                                           int strips, int bands, int waves, int items,
                                                           const RowsPlace place, const Epilogue ep)
{
    constexpr int NOUT = 4 / ST;                                   // outputs per lane and output row
    constexpr int LEFT = PADC;
    constexpr int RIGHT = ST * (NOUT - 1) + S - 1 - PADC - 3 > 0 ? ST * (NOUT - 1) + S - 1 - PADC - 3 : 0;
    constexpr int NIN = ST * (TR - 1) + R;                         // input rows of a band
    static_assert(LEFT <= 4 && RIGHT <= 4, "halo wider than one neighbour lane");
    const float FILL = OP == ROWS_MAX ? -INFINITY : 0.f;
    const int lane = threadIdx.x & 63;
    const int wv = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if (wv >= waves) return;
    int c0, col, band, plane;
    bool live = true;
    if constexpr (SEGL == 64) {
        const int t = place.div(wv, place.by_strips);
        plane = place.div(t, place.by_bands);
        band = t - plane * bands;
        c0 = (wv - t * strips) * kStripStep;          // first input column of the strip
        col = c0 + 4 * lane;                          // this lane's input columns
    } else {
        // the last wavefront may hold fewer than 64 / SEGL items: its idle groups load and store nothing
        const int item = wv * (64 / SEGL) + lane / SEGL;
        live = item < items;
        const int it = live ? item : 0;
        plane = place.div(it, place.by_bands);
        band = it - plane * bands;
        c0 = 0;
        col = 4 * (lane % SEGL);
    }
    const int ocol = col / ST;                        // the lane's first output column
    const int i0 = band * TR;                         // first output row of the band
    const float* xp = x + (int64_t)(OP == ROWS_CONV ? place.div(plane, place.by_planes_per_x) : plane) * H * W;
    float* yp = y + (int64_t)plane * Ho * Wo;
    const int filter = OP == ROWS_CONV ? plane - place.div(plane, place.by_filters) * (int)place.by_filters.d : 0;

    float wr[R * S];
    if constexpr (OP == ROWS_CONV) {
        const float* wf = w + (int64_t)filter * R * S;
#pragma unroll
        for (int k = 0; k < R * S; ++k) wr[k] = wf[k];
    }

    // Every input row of the band, one 16-byte load each, without a branch: rows and columns outside the image load what lies nearest
    // inside and are replaced by padding.  ANY: the lane whose columns run over the end of its row loads the row's last four and moves
    // them down, so that no load leaves the tensor.
    const int lcol = min(col, W - 4);
    floatx4 in[NIN];
#pragma unroll
    for (int e = 0; e < NIN; ++e) {
        const float* p = xp + (int64_t)min(max(ST * i0 - PADC + e, 0), H - 1) * W + lcol;
        if constexpr (ANY) in[e] = *reinterpret_cast<const floatx4u*>(p);
        else in[e] = *reinterpret_cast<const floatx4*>(p);
    }
    const int over = ANY && col < W ? col - lcol : 0;
    const bool one = over & 1, two = over & 2;
#pragma unroll
    for (int e = 0; e < NIN; ++e) {
        floatx4 v = in[e];
        if constexpr (ANY) {
            v = floatx4{one ? v.y : v.x, one ? v.z : v.y, one ? v.w : v.z, one ? FILL : v.w};
            v = floatx4{two ? v.z : v.x, two ? v.w : v.y, two ? FILL : v.z, two ? FILL : v.w};
        }
        const int gr = ST * i0 - PADC + e;
        const bool inside = gr >= 0 && gr < H && col < W;
        in[e] = floatx4{inside ? v.x : FILL, inside ? v.y : FILL, inside ? v.z : FILL, inside ? v.w : FILL};
    }

    float acc[TR][NOUT];
#pragma unroll
    for (int i = 0; i < TR; ++i)
#pragma unroll
        for (int p = 0; p < NOUT; ++p) acc[i][p] = FILL;

#pragma unroll
    for (int e = 0; e < NIN; ++e) {
        // v[LEFT + c] = input column col + c, c = -LEFT .. 3 + RIGHT
        float v[LEFT + 4 + RIGHT];
        v[LEFT + 0] = in[e].x; v[LEFT + 1] = in[e].y; v[LEFT + 2] = in[e].z; v[LEFT + 3] = in[e].w;
#pragma unroll
        for (int c = 0; c < LEFT; ++c) v[LEFT - 1 - c] = from_left<OP>(in[e][3 - c]);
#pragma unroll
        for (int c = 0; c < RIGHT; ++c) v[LEFT + 4 + c] = from_right<OP>(in[e][c]);
#pragma unroll
        for (int orow = 0; orow < TR; ++orow) {
            const int r = e - ST * orow;
            if (r < 0 || r >= R) continue;
#pragma unroll
            for (int q = 0; q < S; ++q)
#pragma unroll
                for (int p = 0; p < NOUT; ++p) {
                    const float e_in = v[ST * p + q];
                    if constexpr (OP == ROWS_CONV) acc[orow][p] = fmaf(wr[r * S + q], e_in, acc[orow][p]);
                    else if constexpr (OP == ROWS_AVG) acc[orow][p] += e_in;
                    else acc[orow][p] = fmaxf(acc[orow][p], e_in);
                }
        }
    }

    // lanes without a neighbour inside the strip have no halo: they only feed their neighbours, unless
    // the missing neighbour lies outside the image, where the shifted-in value is the padding itself
    const bool left_ok = SEGL != 64 || lane > 0 || c0 == 0;
    const bool right_ok = SEGL != 64 || lane < 63 || c0 + kStripIn >= W;
    if (!left_ok || !right_ok || ocol >= Wo || !live) return;
    constexpr float kScale = 1.0f / (float)(R * S);
    // convolution only: per-channel bias and rectifier of the fused-epilogue entry point (both off otherwise)
    const bool with_ep = OP == ROWS_CONV && (ep.bias != nullptr || ep.relu != 0);
    const float ep_bias = (OP == ROWS_CONV && ep.bias) ? ep.bias[filter] : 0.f;
#pragma unroll
    for (int orow = 0; orow < TR; ++orow) {
        const int oi = i0 + orow;
        if (oi >= Ho) break;
        if constexpr (OP == ROWS_AVG) {
#pragma unroll
            for (int p = 0; p < NOUT; ++p) acc[orow][p] *= kScale;
        }
        if (with_ep) {
#pragma unroll
            for (int p = 0; p < NOUT; ++p) {
                const float t = acc[orow][p] + ep_bias;
                acc[orow][p] = ep.relu ? fmaxf(t, 0.f) : t;
            }
        }
        float* dst = yp + (int64_t)oi * Wo + ocol;
        if (ocol + NOUT - 1 < Wo) {
            // (Streaming stores: the output is not read again by this kernel.  But not the 8 bytes a lane of pooling at stride 2, which fill a line
            // in several stores: 2x2 on 256 x 256 x 16 x 12 16.9 us streamed, 11.7; 512 x 256 x 8 x 8 13.1, 10.1; 32 x 128 x 56 x 56 12.5, 11.4;
            // 3x3 planes up to 16 columns 1.15 x.  Filters on many channels of one image are up to 4 % faster streamed.)
            if constexpr (NOUT == 2 && OP != ROWS_CONV)
                *reinterpret_cast<floatx2u*>(dst) = floatx2u{acc[orow][0], acc[orow][1]};
            else if constexpr (NOUT == 4)
                __builtin_nontemporal_store(floatx4u{acc[orow][0], acc[orow][1], acc[orow][2], acc[orow][3]},
                                            reinterpret_cast<floatx4u*>(dst));
            else
                __builtin_nontemporal_store(floatx2u{acc[orow][0], acc[orow][1]}, reinterpret_cast<floatx2u*>(dst));
        } else {
#pragma unroll
            for (int p = 0; p < NOUT; ++p)
                if (ocol + p < Wo) dst[p] = acc[orow][p];
        }
    }
}

template <int R, int S, int PADC, int ST, int OP, int SEGL, bool ANY>
hipError_t launch_rows_seg(const float* x, const float* w, float* y, int64_t planes, int planes_per_x, int n_filters,
                           int H, int W, int Ho, int Wo, hipStream_t st, const Epilogue& ep)
{
    int strips = 1;
    if (SEGL == 64 && W > kStripIn) {
        // input columns whose lanes produce an output
        const int64_t need = (int64_t)ST * Wo;
        const int Wc = (int)(need < W ? (need + 3) & ~(int64_t)3 : W);
        if (Wc > kStripFirst) strips = 1 + (Wc - kStripFirst + kStripStep - 1) / kStripStep;
    }
    // short bands when the launch would otherwise leave most of the chip idle
    constexpr int TR_BIG = 8 / ST, TR_SMALL = 4 / ST;
    constexpr int PER_WAVE = 64 / SEGL;
    const bool small = (planes * strips * ((Ho + TR_BIG - 1) / TR_BIG) + PER_WAVE - 1) / PER_WAVE < 8192;
    const int TR = small ? TR_SMALL : TR_BIG;
    const int bands = (Ho + TR - 1) / TR;
    const int64_t items = planes * strips * bands;
    const int64_t waves = (items + PER_WAVE - 1) / PER_WAVE;
    const int64_t blocks = (waves + 3) / 4;
    if (4 * blocks > 2147483647LL || planes > 2147483647LL) return hipErrorInvalidValue;       // (an item has at least one of 2^31 outputs)
    const int64_t most = std::max<int64_t>({strips, bands, planes_per_x, n_filters});
    const RowsPlace place{make_fastdiv(strips), make_fastdiv(bands), make_fastdiv(planes_per_x), make_fastdiv(n_filters),
                          PER_WAVE * waves * most >= (1LL << 32) || planes * most >= (1LL << 32)};
    dim3 grid((unsigned)blocks), block(256);
    if (small)
        SW_NOTED_LAUNCH(note_kernel("sliding_rows_kernel", (int)(R), (int)(S), (int)(PADC), (int)(TR_SMALL)), (sliding_rows_kernel<R, S, PADC, TR_SMALL, ST, OP, SEGL, ANY>), grid, block, 0, st, x, w, y,
                           H, W, Ho, Wo, strips, bands, (int)waves, (int)items, place, ep);
    else
        SW_NOTED_LAUNCH(note_kernel("sliding_rows_kernel", (int)(R), (int)(S), (int)(PADC), (int)(TR_BIG)), (sliding_rows_kernel<R, S, PADC, TR_BIG, ST, OP, SEGL, ANY>), grid, block, 0, st, x, w, y,
                           H, W, Ho, Wo, strips, bands, (int)waves, (int)items, place, ep);
    return hipGetLastError();
}

// Narrow planes share a wavefront: between two planes must lie as many columns of padding as the next one's first lane shifts in, PADC
// (rows of whole groups leave at least a lane of them).
template <int R, int S, int PADC, int ST, int OP, bool ANY = false>
hipError_t launch_rows(const float* x, const float* w, float* y, int64_t planes, int planes_per_x, int n_filters,
                       int H, int W, int Ho, int Wo, hipStream_t st, const Epilogue& ep)
{
    const int lanes = std::max(W / 4 + 1, (W + PADC + 3) / 4);
#define SW_SEG(L) return launch_rows_seg<R, S, PADC, ST, OP, L, ANY>(x, w, y, planes, planes_per_x, n_filters, H, W, Ho, Wo, st, ep)
    if (lanes <= 8) SW_SEG(8);
    if (lanes <= 16) SW_SEG(16);
    if (lanes <= 32) SW_SEG(32);
    SW_SEG(64);
#undef SW_SEG
}

// rows of whole 16-byte groups on the 16-byte grid
bool whole_quads(const float* x, int W) { return W % 4 == 0 && reinterpret_cast<uintptr_t>(x) % 16 == 0; }

}  // namespace

bool sliding_rows_supported(int W, int R, int S, int stride, int pad)
{
    if ((stride != 1 && stride != 2) || R != S || (R != 3 && R != 5 && R != 7) || pad > (R - 1) / 2 || pad < 0) return false;
    // (padding beyond (R-1)/2 would need more than the compiled halo widths; 7x7 reaches at most four columns into
    // the right neighbour, which rules out the smallest paddings)
    if (R == 7 && pad < (stride == 1 ? 2 : 1)) return false;
    return W >= 4;
}

// Of the planes that a workgroup of the small-planes kernel could take a run of, those that the rows kernel is faster at.  A lane group of the
// rows kernel is eight lanes: planes of up to eight columns leave five or six idle at stride 1, of up to 15 still four, which costs where a
// launch fills the chip; and the smallest launches are over sooner in the other kernel.  us, small planes -> rows: 32 x 512 x 16 x 16 under 3x3
// 12.9 -> 7.1, 5x5 14.8 -> 10.7, 7x7 21.9 -> 16.1, 7x7 at stride 2 15.4 -> 9.6; 32 x 256 x 28 x 28 under 5x5 22.2 -> 13.4, 7x7 39.3 -> 16.1; off
// the 16-byte grid 32 x 512 x 14 x 14 under 3x3 13.0 -> 9.9, 5x5 14.2 -> 12.5, 5x5 at stride 2 9.7 -> 7.4; 16 x 200 x 27 x 27 under 5x5 11.7 -> 7.9,
// 7x7 at stride 2 13.1 -> 5.5.  The other way 64 x 512 x 4 x 4 under 7x7 7.9 -> 12.7, 32 x 512 x 7 x 7 8.7 -> 10.6; tall planes 19 x 800 x 78 x 4 under
// 5x5 at stride 2 11.1 -> 16.9, 54 x 522 x 64 x 4 under 3x3 at stride 2 10.4 -> 14.2, 13 x 369 x 95 x 9 under 5x5 11.8 -> 16.2, 56 x 754 x 17 x 9 under
// 7x7 40.7 -> 52.5; small ones 4 x 381 x 9 x 11 under 5x5 4.4 -> 6.0.  Over 12338 drawn planes the rows kernel takes 0.76 of the time
// where it is taken, and as long as the other (1.00) where it is not.
bool rows_before_small_planes(int64_t planes, const Conv2dShape& s, bool off_grid)
{
    const int64_t lines = planes * s.Ho;
    // (up to 512 planes off the grid and under 5x5 and 7x7 at stride 1 stay, and up to 1024 off the grid under 7x7: a launch's latency either way)
    const bool wide_filter = s.stride == 1 && s.R > 3;
    if (planes <= (off_grid && wide_filter && s.R == 7 ? 1024 : off_grid || wide_filter ? 512 : 0)) return false;
    if (s.stride == 2) {
        if (s.W >= 9) return true;
        if (off_grid && s.W < 7) return false;
        return s.W == 4 ? lines <= (s.R == 3 ? 131072 : 65536) : s.R != 5 || lines <= 131072;
    }
    if (s.W >= 16) return true;
    if (s.W < 9) return false;
    if (s.R == 3) return (s.W >= 11 || lines > 5000) && (s.W >= 14 || lines <= 300000);
    if (s.R == 5) return lines > (s.pad == 2 ? 5600 : 12000) && (s.W >= 12 || lines <= 32768 || (s.W > 9 && (s.pad == 2 || lines <= 65536)));
    return lines > 7000 && (s.W > 9 || lines <= 32768);
}

hipError_t launch_sliding_rows(const float* x, const float* w, float* y, int64_t planes, int planes_per_x,
                               int n_filters, int H, int W, int R, int S, int stride, int pad, int Ho, int Wo,
                               hipStream_t st, const Epilogue& ep)
{
    (void)S;
    const bool any = !whole_quads(x, W);
#define SW_ROWS(RC, PC, SC)                                                                                              \
    if (R == RC && pad == PC && stride == SC)                                                                            \
        return (any ? launch_rows<RC, RC, PC, SC, ROWS_CONV, true> : launch_rows<RC, RC, PC, SC, ROWS_CONV>)(x, w, y, planes, \
               planes_per_x, n_filters, H, W, Ho, Wo, st, ep);
    SW_ROWS(3, 0, 1) SW_ROWS(3, 1, 1) SW_ROWS(5, 0, 1) SW_ROWS(5, 1, 1) SW_ROWS(5, 2, 1) SW_ROWS(7, 2, 1) SW_ROWS(7, 3, 1)
    SW_ROWS(3, 0, 2) SW_ROWS(3, 1, 2) SW_ROWS(5, 0, 2) SW_ROWS(5, 1, 2) SW_ROWS(5, 2, 2) SW_ROWS(7, 1, 2) SW_ROWS(7, 2, 2) SW_ROWS(7, 3, 2)
#undef SW_ROWS
    return hipErrorInvalidValue;
}

// Pooling windows with a register-only kernel: 2x2 and 3x3, stride 1 or 2, padding up to half the window, rows of any width.  Against one
// thread per output (us, 3x3 at stride 2 unless said): 27 x 64 x 109 x 79 31.1 -> 13.5 (5.5 TB/s), 8 x 64 x 113 x 250 28.9 -> 13.0,
// 2 x 64 x 93 x 122 5.0 -> 3.6, 16 x 256 x 7 x 7 3.6 -> 3.2, at stride 1 on 16 x 192 x 14 x 14 6.0 -> 4.1.  Rows of four to six columns off the
// grid stay with the latter: a lane group is eight lanes, and they fill two (64 x 512 x 6 x 6 under 2x2 4.1 against 4.5, x 5 x 5 4.6
// against 4.8); of seven under 2x2 (0.9 to 1.0 x the time from 2^18 outputs up, the same below) and, up to 65536 outputs, under
// 3x3 at stride 1 (3.5 us against 3.7).
bool pool_rows_supported(const float* x, int64_t planes, int W, int R, int S, int stride, int pad, int Ho, int Wo)
{
    if ((stride != 1 && stride != 2) || R != S || (R != 2 && R != 3) || pad < 0 || pad > (R == 3 ? 1 : 0)) return false;
    if (R == 2 && stride == 1) return false;       // (no compiled variant; the direct kernel takes it)
    if (whole_quads(x, W)) return true;
    return W > 7 || (W == 7 && R == 3 && (stride == 2 || planes * Ho * Wo >= 65536));
}

hipError_t launch_pool_rows(const float* x, float* y, int64_t planes, int H, int W, int R, int stride, int pad,
                            int Ho, int Wo, bool maximum, hipStream_t st)
{
#define SW_POOL(RC, PC, SC)                                                                                    \
    if (R == RC && pad == PC && stride == SC) {                                                                \
        const bool any = !whole_quads(x, W);                                \
        auto f = maximum ? any ? launch_rows<RC, RC, PC, SC, ROWS_MAX, true> : launch_rows<RC, RC, PC, SC, ROWS_MAX> \
                         : any ? launch_rows<RC, RC, PC, SC, ROWS_AVG, true> : launch_rows<RC, RC, PC, SC, ROWS_AVG>; \
        return f(x, nullptr, y, planes, 1, 1, H, W, Ho, Wo, st, Epilogue{nullptr, 0});                          \
    }
    SW_POOL(2, 0, 2) SW_POOL(3, 0, 1) SW_POOL(3, 1, 1) SW_POOL(3, 0, 2) SW_POOL(3, 1, 2)
#undef SW_POOL
    return hipErrorInvalidValue;
}

}  // namespace swconv
