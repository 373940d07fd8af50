// One filter per plane (depthwise, or one input channel) over planes of any width: bands of output rows, fp32 or bf16 planes,
// any filter extent and any stride (paper, section 1.2; section 2: the input is used as it lies in memory).
//
// The register-only rows kernel needs whole 16-byte groups per image row, and the 56 x 56 tile of the sliding kernel stride 1;
// what they refuse ran one thread per output.  Here a workgroup takes a band of output rows of one plane: the input rows it
// touches come into LDS once, framed by their zero padding, four columns at a time (16-byte loads that may start at any
// 4-byte address; columns beside the image are cleared in registers), and a thread owns four consecutive outputs of a column:
// for every filter column it reads the 3 stride + R inputs they depend on once and slides them under the taps by renaming
// registers.  Taps are wave-uniform (scalar registers).  Consecutive threads own consecutive columns: every store instruction
// writes a run of consecutive outputs.
//
// Measured (us per launch, replayed graphs of ten): fp32 5x5 stride 2 on 8 x 144 x 75 x 75 36.1 (one thread per output) -> 9.5,
// 3.4 TB/s; 7x7 on 8 x 488 x 47 x 42 39.7 (tile kernel) -> 26.9; bf16 5x5 stride 2 on 8 x 144 x 75 x 75 31.2 -> 9.7.  Bound by the memory round
// trip in front of each workgroup's only barrier, and by LDS reads for the larger filters (18 per 49 multiply-adds at 7x7).
#include <algorithm>

#include "swconv_internal.h"

namespace swconv {

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr unsigned kBeyond = 0x80000000u;
constexpr int kBandFloats = 6 * 1024;       // 24 KB: six workgroups per CU, so that some load while others compute
constexpr int kBandMax = 16 * 1024;         // a band of four output rows of the widest planes

struct BandParams {
    Epilogue ep;
    int H, W, R, S, stride, pad, Ho, Wo, n_filters, planes_per_x;
    int QH, bands;                          // groups of four output rows per band, bands per plane
    int Wp4, cells4;                        // framed row and framed band in groups of four columns
    unsigned x_bytes;
    FastDiv by_bands, by_Wp4, by_Wo;
};

// RC, STC > 0: filter extent and stride at compile time (taps unrolled); 0: at run time.  BF: bf16 planes.
template <int RC, int STC, bool BF>
__global__ __launch_bounds__(256) void plane_bands_kernel(const void* __restrict__ x, const float* __restrict__ w, void* __restrict__ y,
                                                          const BandParams P)
{
    extern __shared__ __attribute__((aligned(16))) float xs[];         // [framed rows][Wp4 * 4]
    const int R = RC > 0 ? RC : P.R, S = RC > 0 ? RC : P.S, ST = RC > 0 ? STC : P.stride;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int plane = fast_div(blockIdx.x, P.by_bands), band = blockIdx.x - plane * P.bands;
    const int o0 = 4 * P.QH * band;                                    // first output row
    const int px = plane / P.planes_per_x, f = plane % P.n_filters;
    const int h0 = o0 * ST - P.pad;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(x), 0, P.x_bytes, 0x00020000);

    // four groups of four columns in flight per thread
    for (int base = tid; base < P.cells4; base += 4 * nt) {
        floatx4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + u * nt;
            const int hp = fast_div(i, P.by_Wp4), c = 4 * (i - hp * P.Wp4) - P.pad, h = h0 + hp;
            const bool in = i < P.cells4 && h >= 0 && h < P.H && c < P.W && c > -4;
            const int64_t at = ((int64_t)px * P.H + h) * P.W + c;
            if constexpr (BF) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const unsigned bits = __builtin_amdgcn_raw_buffer_load_b16(xr, in && (unsigned)(c + e) < (unsigned)P.W ? (unsigned)((at + e) * 2) : kBeyond, 0, 0);
                    v[u][e] = __uint_as_float(bits << 16);
                }
            } else if (__builtin_expect(in && (at < 0 || (unsigned)(at * 4) + 16u > P.x_bytes), 0)) {
#pragma unroll
                for (int e = 0; e < 4; ++e)         // the first or the last values of the tensor, one by one
                    v[u][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xr, (unsigned)(c + e) < (unsigned)P.W ? (unsigned)((at + e) * 4) : kBeyond, 0, 0));
            } else {
                v[u] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(xr, in ? (unsigned)(at * 4) : kBeyond, 0, 0));
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = base + u * nt;
            if (i >= P.cells4) break;
            const int hp = fast_div(i, P.by_Wp4), c = 4 * (i - hp * P.Wp4) - P.pad;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((unsigned)(c + e) >= (unsigned)P.W) v[u][e] = 0.f;
            reinterpret_cast<floatx4*>(xs)[i] = v[u];
        }
    }
    __syncthreads();

    const int pitch = 4 * P.Wp4;
    const int rows = min(4 * P.QH, P.Ho - o0), items = ((rows + 3) / 4) * P.Wo;
    const float* wf = w + (int64_t)f * R * S;
    const float bias = P.ep.bias ? P.ep.bias[f] : 0.f;
    for (int idx = tid; idx < items; idx += nt) {
        const int q4 = fast_div(idx, P.by_Wo), oj = idx - q4 * P.Wo;
        const float* xp = xs + 4 * q4 * ST * pitch + oj * ST;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (RC > 0) {
            constexpr int N = 3 * STC + RC;         // inputs of a filter column that the four outputs touch
            float odd[4] = {0.f, 0.f, 0.f, 0.f};    // every second column apart: shorter sums, smaller rounding errors
#pragma unroll
            for (int q = 0; q < RC; ++q) {
                float in[N];
#pragma unroll
                for (int c = 0; c < N; ++c) in[c] = xp[c * pitch + q];
#pragma unroll
                for (int r = 0; r < RC; ++r) {
                    const float tap = wf[r * RC + q];
#pragma unroll
                    for (int j = 0; j < 4; ++j) (q & 1 ? odd : acc)[j] = fmaf(tap, in[j * STC + r], (q & 1 ? odd : acc)[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] += odd[j];
        } else {
            for (int r = 0; r < R; ++r)
                for (int q = 0; q < S; ++q) {
                    const float tap = wf[r * S + q];
                    const float* col = xp + r * pitch + q;
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[j] = fmaf(tap, col[j * ST * pitch], acc[j]);
                }
        }
        const int oi = o0 + 4 * q4;
        const int64_t at = ((int64_t)plane * P.Ho + oi) * P.Wo + oj;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (oi + j >= P.Ho) break;
            float t = acc[j];
            if (P.ep.bias) t += bias;
            if (P.ep.relu) t = fmaxf(t, 0.f);
            if constexpr (BF) reinterpret_cast<__bf16*>(y)[at + j * P.Wo] = (__bf16)t;
            else reinterpret_cast<float*>(y)[at + j * P.Wo] = t;
        }
    }
}

struct BandPlan {
    bool ok = false;
    int threads = 256;
    int64_t groups = 0;
    BandParams P;
};

BandPlan plan_bands(const void* x, int64_t planes, int planes_per_x, int n_filters, const Conv2dShape& s, int bytes)
{
    BandPlan a;
    const int64_t x_bytes = ((planes + planes_per_x - 1) / planes_per_x) * s.H * s.W * bytes;
    if (s.dil != 1 || x_bytes >= (1LL << 31) || reinterpret_cast<uintptr_t>(x) % bytes != 0) return a;
    const int64_t Wp4 = ((int64_t)(s.Wo - 1) * s.stride + s.S + 3) / 4;
    const int QHall = (s.Ho + 3) / 4;
    const auto floats = [&](int64_t qh) { return ((4 * qh - 1) * s.stride + s.R) * 4 * Wp4; };
    if (floats(1) > kBandMax) return a;
    int QH = 1;
    while (QH < QHall && floats(QH + 1) <= kBandFloats) ++QH;
    int bands = (QHall + QH - 1) / QH;
    while (planes * bands < 768 && bands < QHall) ++bands;     // enough workgroups for the chip before the bands grow
    QH = (QHall + bands - 1) / bands;
    bands = (QHall + QH - 1) / QH;
    if (planes * bands * bands >= (1LL << 31)) return a;
    a.groups = planes * bands;
    a.threads = (int64_t)QH * s.Wo <= 128 ? 128 : 256;
    if (a.groups * a.threads >= (1LL << 32)) return a;      // (work items of a launch)
    a.ok = true;
    BandParams& P = a.P;
    P.H = s.H; P.W = s.W; P.R = s.R; P.S = s.S; P.stride = s.stride; P.pad = s.pad; P.Ho = s.Ho; P.Wo = s.Wo;
    P.n_filters = n_filters; P.planes_per_x = planes_per_x;
    P.QH = QH; P.bands = bands;
    P.Wp4 = (int)Wp4; P.cells4 = (int)(floats(QH) / 4);
    P.x_bytes = (unsigned)x_bytes;
    P.by_bands = make_fastdiv(bands); P.by_Wp4 = make_fastdiv((int)Wp4); P.by_Wo = make_fastdiv(s.Wo);
    return a;
}

template <int RC, int STC, bool BF>
hipError_t launch_bands(const void* x, const float* w, void* y, const BandPlan& a, hipStream_t st)
{
    const size_t lds = (size_t)a.P.cells4 * 16;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(plane_bands_kernel<RC, STC, BF>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kBandMax * 4);
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel("plane_bands_kernel", RC, STC, BF), (plane_bands_kernel<RC, STC, BF>), dim3((unsigned)a.groups), dim3(a.threads), lds,
                    st, x, w, y, a.P);
    return hipGetLastError();
}

template <bool BF>
hipError_t launch_any(const void* x, const float* w, void* y, const BandPlan& a, hipStream_t st)
{
    const BandParams& P = a.P;
    if (P.R == P.S && P.stride == 1) {
        if (P.R == 3) return launch_bands<3, 1, BF>(x, w, y, a, st);
        if (P.R == 5) return launch_bands<5, 1, BF>(x, w, y, a, st);
        if (P.R == 7) return launch_bands<7, 1, BF>(x, w, y, a, st);
    }
    if (P.R == P.S && P.stride == 2) {
        if (P.R == 3) return launch_bands<3, 2, BF>(x, w, y, a, st);
        if (P.R == 5) return launch_bands<5, 2, BF>(x, w, y, a, st);
        if (P.R == 7) return launch_bands<7, 2, BF>(x, w, y, a, st);
    }
    return launch_bands<0, 0, BF>(x, w, y, a, st);
}

}  // namespace

// Where bands are no slower than one thread per output.  us, one thread per output / bands:
// - Taps unrolled: a workgroup per plane needs enough to do.  131072 planes under 3x3, 81 outputs each, 59.6 / 74.5, 121 outputs 86.3 /
//   74.9; 5x5, 49 outputs 66.9 / 84.2, 81 outputs 109 / 85.5; 7x7 stride 2, 25 outputs 109 / 131, 36 outputs 133 / 133.  With few planes
//   bands were never slower (256 planes under 3x3, 25 outputs each, 3.93 / 3.98; 4096 under 5x5, 49 outputs each, 6.7 / 5.8).
// - Taps in loops: bands pay for the framed plane and for whole groups of four output rows, one thread per output for the taps that
//   meet the plane (`met`: at most R / stride rows of taps meet an input row).  The lines fit 845 timed shapes; six lie on the wrong
//   side by more than 6 %, at most 17 %.  113 x 113, 512 planes: 2x2 stride 4 5.0 / 8.4, 3x3 stride 4 7.1 / 8.7, stride 3 10.0 / 8.7,
//   7x7 stride 8 16.1 / 10.5, 256 planes: 9x9 stride 4 25.0 / 11.7, 51x51 stride 3 602 / 461; 6x6 stride 9 on 225 x 84 23.4 / 27.8; 33x33 on 12 x 5, mostly over the padding,
//   44 / 83; 21x21 stride 7 on 23 x 230, one output row, 63 / 119; 2x2 on 8 planes of 118 x 279 3.5 / 4.1.
bool plane_bands_worthwhile(int64_t planes, const Conv2dShape& s, bool bf16)
{
    const int taps = s.R * s.S;
    const int64_t work = (int64_t)s.Ho * s.Wo * taps;
    if (bf16 && work < 2000) return false;      // (3x3 stride 2 on 19 x 19: 3.5 us against 3.8; 7x7 on 10 x 10: 8.0 against 11.9)
    if (plane_bands_unrolled(s)) return bf16 || planes <= (s.R == 3 ? 512 : 4096) || work >= (s.R == 3 ? 1000 : 1600);
    const auto met = [&](int n, int k, int n_out) { return std::min((double)n_out * k, n * std::min((double)n_out, (double)k / s.stride)); };
    const double real = met(s.H, s.R, s.Ho) * met(s.W, s.S, s.Wo);
    const double frame = ((double)(s.Ho - 1) * s.stride + s.R) * ((double)(s.Wo - 1) * s.stride + s.S);
    const bool few = planes <= 512;
    if ((few ? 4 : 3) * real < (double)((s.Ho + 3) / 4 * 4) * s.Wo * taps) return false;
    if (few && taps >= (bf16 ? 25 : 12) && real >= frame) return true;
    if (taps < 25) return (double)planes * real >= 1e6 && real >= frame + 1000;
    return real >= (bf16 ? frame : frame / 2) + 2000;
}

bool plane_bands_supported(const void* x, int64_t planes, int planes_per_x, int n_filters, const Conv2dShape& s, bool bf16)
{
    return plane_bands_worthwhile(planes, s, bf16) && plan_bands(x, planes, planes_per_x, n_filters, s, bf16 ? 2 : 4).ok;
}

hipError_t launch_plane_bands(const void* x, const float* w, void* y, int64_t planes, int planes_per_x, int n_filters, const Conv2dShape& s,
                              bool bf16, hipStream_t st, const Epilogue& ep)
{
    BandPlan a = plan_bands(x, planes, planes_per_x, n_filters, s, bf16 ? 2 : 4);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.ep = ep;
    return bf16 ? launch_any<true>(x, w, y, a, st) : launch_any<false>(x, w, y, a, st);
}

}  // namespace swconv
