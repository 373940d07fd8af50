// C ABI of libswconv.so: host-side validation and kernel selection.  Every argument error is
// reported before anything is enqueued; nothing here allocates device memory or synchronises (the host memory of a thread's launch plans
// is PlanCache's).
#include "../../include/swconv.h"

#include <cstdio>
#include <cstdlib>

#include "swconv_internal.h"

using namespace swconv;

namespace swconv {

namespace {
struct LastKernel {
    const char* name;
    int arg[4];
};
thread_local LastKernel g_last_kernel{nullptr, {-1, -1, -1, -1}};
}  // namespace

void note_kernel(const char* name, int a, int b, int c, int d) { g_last_kernel = LastKernel{name, {a, b, c, d}}; }

}  // namespace swconv

namespace {

constexpr int64_t kMaxElems = 2147483647LL;  // element count per tensor
constexpr int kMaxTaps1D = 64;
constexpr int kMaxFilter2D = 64;

bool force_direct()
{
    static const bool v = [] {
        const char* e = std::getenv("SWCONV_FORCE_DIRECT");
        return e && e[0] == '1';
    }();
    return v;
}

bool misaligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) != 0; }

bool overlaps(const void* a, int64_t abytes, const void* b, int64_t bbytes)
{
    const uintptr_t a0 = reinterpret_cast<uintptr_t>(a), b0 = reinterpret_cast<uintptr_t>(b);
    return a0 < b0 + (uintptr_t)bbytes && b0 < a0 + (uintptr_t)abytes;
}

int launch_status(hipError_t e) { return e == hipSuccess ? SW_OK : SW_ERR_LAUNCH; }

// One filter per plane (single input channel, depthwise): picks among the whole-plane kernel (many planes
// that fit a 56 x 56 tile), the register-only rows kernel (3x3 / 5x5), the tile kernel and the direct kernel.
int run_plane(const float* x, const float* w, float* y, int64_t planes, int planes_per_x, int n_filters,
              const Conv2dShape& s, bool depthwise, hipStream_t st, const Epilogue& ep = Epilogue{nullptr, 0})
{
    if (!force_direct() && s.dil != 1) {
        // dilated taps: the run-time-extent tile kernel, whose window holds the filter's span
        if (sliding_plane_supported(s.H, s.W, s.R, s.S, s.stride, s.pad, s.dil) &&
            sliding_plane_worthwhile(planes, s.Ho, s.Wo, s.R, s.S))
            return launch_status(launch_sliding_plane(x, w, y, planes, planes_per_x, n_filters, s.H, s.W, s.R, s.S,
                                                      s.pad, s.Ho, s.Wo, st, ep, s.dil));
    } else if (!force_direct()) {
        const bool off_grid = s.W % 4 != 0 || misaligned(x, 16);
        const bool any_rows = sliding_rows_supported(s.W, s.R, s.S, s.stride, s.pad), rows = any_rows && !off_grid;
        // planes up to 20 x 20, larger filters' planes and larger ragged ones (width not a multiple of 4): a run of planes per workgroup ...
        const bool small = (s.H * s.W <= 400 || s.W % 4 != 0 || s.R * s.S >= 25) &&
                           small_planes_supported(planes, planes_per_x, s.H, s.W, s.R, s.S, s.stride, s.Ho, s.Wo);
        // ... but the rows kernel first where it has a variant and is faster
        if (small && any_rows && rows_before_small_planes(planes, s, off_grid))
            return launch_status(launch_sliding_rows(x, w, y, planes, planes_per_x, n_filters, s.H, s.W, s.R, s.S,
                                                     s.stride, s.pad, s.Ho, s.Wo, st, ep));
        if (small)
            return launch_status(launch_small_planes(x, w, y, planes, n_filters, s.H, s.W, s.R, s.S, s.stride, s.pad,
                                                     s.Ho, s.Wo, st, ep));
        // The whole-plane kernel spends a 56 x 56 tile per plane: less than that leaves lanes idle, and up to 1024 planes do not fill the
        // chip with it; both go to the rows kernel when that has a variant.  us, tile -> rows: 8 x 256 x 48 x 40 under 3x3 12.7 -> 7.2, 7x7
        // 19.5 -> 12.6; 32 x 256 x 48 x 48 5x5 36.0 -> 29.2, 7x7 48.3 -> 43.0; 32 x 256 x 56 x 40 5x5 35.5 -> 31.3; 8 x 64 x 56 x 56 3x3 5.7 -> 4.6,
        // 7x7 9.5 -> 6.5; 16 x 64 x 56 x 56 5x5 8.5 -> 7.1.  It keeps more full planes: 32 x 64 x 56 x 56 under 3x3 10.5 against 11.1, under 5x5
        // 12.4 against 12.6, 128 x 64 under 7x7 49.9 against 54.7.
        const bool whole = s.stride == 1 && sliding_plane_whole(x, y, s.H, s.W, s.R, s.S, s.pad, s.Ho, s.Wo) &&
                           planes >= 512 && !(rows && (s.H < 56 || s.W < 56 || planes <= 1024));
        if (!whole && rows)
            return launch_status(launch_sliding_rows(x, w, y, planes, planes_per_x, n_filters, s.H, s.W, s.R, s.S,
                                                     s.stride, s.pad, s.Ho, s.Wo, st, ep));
        // Bands of output rows, unrolled for 3x3, 5x5 and 7x7 at strides 1 and 2: faster than the 56 x 56 tile per wavefront on
        // every layer timed that reaches this point (us: 8 x 64 x 113 x 113 3x3 26.5 -> 14.8, 8 x 64 x 57 x 57 7x7 24.2 -> 9.8,
        // 8 x 488 x 47 x 42 7x7 39.7 -> 26.9, one image 200 x 62 x 62 3x3 12.2 -> 5.2); the tile keeps the other extents.
        if (!whole && plane_bands_unrolled(s) && plane_bands_supported(x, planes, planes_per_x, n_filters, s, false))
            return launch_status(launch_plane_bands(x, w, y, planes, planes_per_x, n_filters, s, false, st, ep));
        // (where a plane is too little for a workgroup of bands, it is for a tile: 131072 planes of 5 x 5 under 3x3 266 us on tiles, 73 on
        // bands, 22 with one thread per output)
        const bool little = plane_bands_unrolled(s) && !plane_bands_worthwhile(planes, s, false);
        if (!little && sliding_plane_supported(s.H, s.W, s.R, s.S, s.stride, s.pad) &&
            sliding_plane_worthwhile(planes, s.Ho, s.Wo, s.R, s.S))
            return launch_status(launch_sliding_plane(x, w, y, planes, planes_per_x, n_filters, s.H, s.W, s.R, s.S,
                                                      s.pad, s.Ho, s.Wo, st, ep));
    }
    // strides above 1 the rows kernel does not take, few or short planes: bands too, their taps in loops where not unrolled (us:
    // 8 x 144 x 75 x 75 5x5 stride 2 36.1 -> 9.5 in place of one thread per output; plane_bands_worthwhile)
    if (!force_direct() && plane_bands_supported(x, planes, planes_per_x, n_filters, s, false))
        return launch_status(launch_plane_bands(x, w, y, planes, planes_per_x, n_filters, s, false, st, ep));
    return launch_status(launch_direct_conv2d_f32(x, w, y, s, depthwise, st, &ep));
}

// Shared validation of the 2-D calls.  esz_in / esz_out are element sizes in bytes.
int check_conv2d(const void* x, const void* w, const void* y, int N, int C_in, int C_out, int H, int W,
                 int R, int S, int stride, int pad, bool depthwise, size_t esz_in, size_t esz_out,
                 Conv2dShape* out, int dil = 1)
{
    if (!x || !w || !y) return SW_ERR_NULL;
    if (N <= 0 || C_in <= 0 || C_out <= 0 || H <= 0 || W <= 0 || R <= 0 || S <= 0 || stride <= 0 || pad < 0 ||
        dil <= 0)
        return SW_ERR_SHAPE;
    // a dilated filter spans dil * (k - 1) + 1 input positions
    const int64_t span_r = (int64_t)dil * (R - 1) + 1, span_s = (int64_t)dil * (S - 1) + 1;
    if (span_r > kMaxElems || span_s > kMaxElems) return SW_ERR_SHAPE;
    const int64_t Ho = sw_out_dim(H, (int)span_r, stride, pad), Wo = sw_out_dim(W, (int)span_s, stride, pad);
    if (Ho <= 0 || Wo <= 0) return SW_ERR_SHAPE;
    const int64_t nx = (int64_t)N * C_in * H * W;
    const int64_t nw = (int64_t)C_out * (depthwise ? 1 : C_in) * R * S;
    const int64_t ny = (int64_t)N * C_out * Ho * Wo;
    if (nx > kMaxElems || nw > kMaxElems || ny > kMaxElems) return SW_ERR_SHAPE;
    if ((int64_t)H + 2 * (int64_t)pad > kMaxElems || (int64_t)W + 2 * (int64_t)pad > kMaxElems)
        return SW_ERR_SHAPE;
    if (R > kMaxFilter2D || S > kMaxFilter2D) return SW_ERR_UNSUPPORTED;
    if (misaligned(x, esz_in) || misaligned(w, esz_in) || misaligned(y, esz_out)) return SW_ERR_ALIGN;
    if (overlaps(y, ny * (int64_t)esz_out, x, nx * (int64_t)esz_in) ||
        overlaps(y, ny * (int64_t)esz_out, w, nw * (int64_t)esz_in))
        return SW_ERR_ALIAS;
    *out = Conv2dShape{N, C_in, C_out, H, W, R, S, stride, pad, (int)Ho, (int)Wo, dil};
    return SW_OK;
}

int run_1d(const float* x, const float* w, float* y, int64_t rows, int64_t len, int k, int stride, int pad,
           Op1D op, void* hip_stream)
{
    if (!x || !y || (op == OP_CONV && !w)) return SW_ERR_NULL;
    if (rows <= 0 || len <= 0 || k <= 0 || stride <= 0 || pad < 0) return SW_ERR_SHAPE;
    const int64_t len_out = sw_out_dim(len, k, stride, pad);
    if (len_out <= 0) return SW_ERR_SHAPE;
    if (len > kMaxElems / rows || len_out > kMaxElems / rows) return SW_ERR_SHAPE;
    if (k > kMaxTaps1D || pad >= k) return SW_ERR_UNSUPPORTED;
    if (misaligned(x, 4) || misaligned(y, 4) || (w && misaligned(w, 4))) return SW_ERR_ALIGN;
    if (overlaps(y, rows * len_out * 4, x, rows * len * 4) || (w && overlaps(y, rows * len_out * 4, w, k * 4)))
        return SW_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (!force_direct() && sliding_1d_supported(len, k, stride, pad))
        return launch_status(launch_sliding_1d(x, w, y, rows, len, len_out, k, pad, op, st));
    if (!force_direct() && op != OP_CONV && pool_tiles_supported(x, y, len, k, stride))
        return launch_status(launch_pool_tiles(x, y, rows, len, k, op == OP_MAX, st));
    if (!force_direct() && strided_1d_supported(rows, len, len_out, k, stride, pad))
        return launch_status(launch_strided_1d(x, w, y, rows, len, len_out, k, stride, pad, op, st));
    return launch_status(launch_direct_1d(x, w, y, rows, len, len_out, k, stride, pad, op, st));
}

}  // namespace

extern "C" {

int64_t sw_out_dim(int64_t in, int k, int stride, int pad)
{
    if (in <= 0 || k <= 0 || stride <= 0 || pad < 0) return 0;
    const int64_t span = in + 2 * (int64_t)pad - k;
    if (span < 0) return 0;
    return span / stride + 1;
}

int64_t sw_out_dim_dilated(int64_t in, int k, int stride, int pad, int dilation)
{
    if (k <= 0 || dilation <= 0) return 0;
    const int64_t span = (int64_t)dilation * (k - 1) + 1;      // input positions a dilated filter covers
    if (span > kMaxElems) return 0;
    return sw_out_dim(in, (int)span, stride, pad);
}

size_t sw_workspace_bytes(void) { return 0; }

const char* sw_status_string(int status)
{
    switch (status) {
        case SW_OK: return "ok";
        case SW_ERR_NULL: return "a required pointer is NULL";
        case SW_ERR_SHAPE: return "invalid shape, stride or padding";
        case SW_ERR_UNSUPPORTED: return "valid problem without a kernel in this library";
        case SW_ERR_ALIGN: return "pointer not aligned to its element size";
        case SW_ERR_ALIAS: return "output overlaps an input";
        case SW_ERR_LAUNCH: return "HIP launch failed";
        case SW_ERR_JIT: return "run-time compilation of a generated kernel failed";
        default: return "unknown status";
    }
}

int sw_version(void) { return 200; }

const char* sw_last_kernel(void)
{
    thread_local char text[160];
    const auto& k = g_last_kernel;
    if (!k.name) return "";
    int n = std::snprintf(text, sizeof text, "%s", k.name);
    for (int i = 0; i < 4 && k.arg[i] >= 0 && n > 0 && n < (int)sizeof text; ++i)
        n += std::snprintf(text + n, sizeof text - n, "%s%d", i == 0 ? "<" : ",", k.arg[i]);
    if (k.arg[0] >= 0 && n > 0 && n < (int)sizeof text - 1) std::snprintf(text + n, sizeof text - n, ">");
    return text;
}

int sw_conv1d(const float* x, const float* w, float* y, int64_t rows, int64_t len, int k, int stride,
              int pad, void* hip_stream)
{
    return run_1d(x, w, y, rows, len, k, stride, pad, OP_CONV, hip_stream);
}

int sw_pool1d(const float* x, float* y, int64_t rows, int64_t len, int window, int stride, int mode,
              void* hip_stream)
{
    if (mode != SW_POOL_AVG && mode != SW_POOL_MAX) return x && y ? SW_ERR_UNSUPPORTED : SW_ERR_NULL;
    return run_1d(x, nullptr, y, rows, len, window, stride, 0, mode == SW_POOL_AVG ? OP_AVG : OP_MAX,
                  hip_stream);
}

int sw_pool2d(const float* x, float* y, int N, int C, int H, int W, int R, int S, int stride, int pad, int mode,
              void* hip_stream)
{
    if (!x || !y) return SW_ERR_NULL;
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || R <= 0 || S <= 0 || stride <= 0 || pad < 0) return SW_ERR_SHAPE;
    const int64_t Ho = sw_out_dim(H, R, stride, pad), Wo = sw_out_dim(W, S, stride, pad);
    if (Ho <= 0 || Wo <= 0) return SW_ERR_SHAPE;
    const int64_t planes = (int64_t)N * C;
    const int64_t nx = planes * H * W, ny = planes * Ho * Wo;
    if (nx > kMaxElems || ny > kMaxElems) return SW_ERR_SHAPE;
    if (mode != SW_POOL_AVG && mode != SW_POOL_MAX) return SW_ERR_UNSUPPORTED;
    if (R > kMaxFilter2D || S > kMaxFilter2D) return SW_ERR_UNSUPPORTED;
    if (2 * pad > (R < S ? R : S)) return SW_ERR_UNSUPPORTED;   // a window could lie wholly in the padding
    if (misaligned(x, 4) || misaligned(y, 4)) return SW_ERR_ALIGN;
    if (overlaps(y, ny * 4, x, nx * 4)) return SW_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const bool maximum = mode == SW_POOL_MAX;
    if (!force_direct() && global_pool_supported(H, W, R, S, pad))
        return launch_status(launch_global_pool(x, y, planes, H * W, maximum, st));
    if (!force_direct() && pool_rows_supported(x, planes, W, R, S, stride, pad, (int)Ho, (int)Wo))
        return launch_status(launch_pool_rows(x, y, planes, H, W, R, stride, pad, (int)Ho, (int)Wo, maximum, st));
    return launch_status(launch_direct_pool2d(x, y, planes, H, W, R, S, stride, pad, (int)Ho, (int)Wo, maximum, st));
}

// Launches of few tiles (of 16 channels x 16 pixels of an image), whose products the few-tiles kernel spreads over the wavefronts of a
// workgroup.  The lines are where it and the kernels of before cross, on 820 layers drawn over 7 ... 112 pixels, 9 ... 512 channels, 1 x 1 ...
// 7 x 7, strides 1 and 2: nine taps on split operands up to 512 tiles where the two plans' estimates say so (1.04 to 2.4 x taken, 0.4 to 1.1 x
// beyond), 25 and more taps 1.3 to 38 x up to the largest tried (18020), the rest 1.1 to 5 x up to 2048 and 0.9 to 1.1 x up to 3000.
// 25 and more taps over two to six channels are short sums, which the any-shape kernel is as fast at once its launch is filled: 13 x 2 -> 51 at
// 157 x 31 under 5x5 12.9 us there against 27.1 (13468 tiles), 2 x 2 -> 24 at 198 x 329 under 6x6 24.2 against 31.1; of 5904 drawn layers of
// 3000 to 16384 tiles those below the lines are 2.0 x as fast here, those beyond 1.0.
static bool few_tiles(const Conv2dShape& s)
{
    const int64_t tiles = (int64_t)s.N * (((int64_t)s.Ho * s.Wo + 15) / 16) * ((s.C_out + 15) / 16);
    if (s.R * s.S == 9 && mfma_f32_split_supported(s))
        return tiles <= 512 && mfma_f32_few_supported(s) && mfma_f32_few_estimate(s) < 0.95 * mfma_f32_split_estimate(s);
    int64_t most = s.R * s.S >= 25 ? 16384 : 2048;
    if (s.R * s.S >= 25 && s.C_in <= 6) {
        if (s.C_out > 32) most = s.C_in == 2 ? 3000 : 6000;
        else if (s.C_out > 16 && s.C_in == 2) most = 6000;
    }
    return tiles <= most && mfma_f32_few_supported(s);
}

// Those of filters of 5 x 5 to 7 x 7 over 17 to 64 channels into whole blocks of 16, in place of the compound kernel, which has a workgroup per 256 pixels whatever
// the launch (us, graph of ten, compound kernel / this one: 56 -> 80 at 28 x 28 5x5 stride 2 151.6 / 8.3, 20 x 64 -> 96 at 8 x 8 stride 2 150.1 / 8.5,
// 10 x 64 -> 264 at 20 x 20 160.9 / 72.7, 7 x 24 -> 408 at 32 x 32 88.9 / 55.2, 2 x 63 -> 30 at 40 x 40 7x7 stride 2 343.0 / 11.1; of 22 drawn layers
// 1.5 to 31 x, errors against 64 bits a third).  The lines at 16 and 64 channels and at 16 outputs are not where the kernels cross: beyond them tests assert
// the compound kernel's plans.  Both sides, compound kernel / this one: 4 x 64 -> 29 at 8 x 8 7x7 268 / 10.4 (79 layers 2.8 to 34 x), 11 -> 47 at 44 x 44 5x7
// 59 / 6.5 (271 of 8 to 16 channels 1.6 to 15 x), 2 x 64 -> 10 at 42 x 44 5x7 196 / 9.3 (375 into fewer than 16 outputs 5 to 34 x).
static bool few_tiles_before_rows(const Conv2dShape& s)
{
    return s.R >= 5 && s.S >= 5 && s.R * s.S <= 49 && s.C_in > 16 && s.C_in < (s.R * s.S < 49 ? 65 : 64) && s.C_out >= 16;
}

// ... in place of the kernels that come first in run_conv2d: from 65 input channels up where the pointwise kernel does not have the layer; in its place
// from 48 up, up to 640 tiles, or 1600 of 64 and more channels into 128 and more.  Graph of ten, us: 456 -> 48 at 38 x 38, 2 images 20.5 -> 13.4, 272 -> 16
// at 16 x 16, 20 images 13.7 -> 7.3, 64 -> 40 at 36 x 36, 2 images 9.9 -> 5.7, 488 -> 120 at 24 x 24, 3 images 23.0 -> 9.6, 56 -> 104 at 20 x 20, 3
// images 6.8 -> 5.8; of 46 drawn layers up to 640 tiles 1.1 to 3.2 x, of 24 of 800 to 1600 tiles into 128 and more channels 1.1 to 2.0 x, errors against 64 bits
// smaller in each.  Beyond it is 0.85 to 1.25 x, into fewer channels 0.5 (144 -> 16 at 68 x 68, 7 images) to 1.6 x, and from fewer 0.8 to 1.3 x.  The lines at 48
// channels and 128 tiles are not where the kernels cross: tests assert the pointwise kernel's plans there.  Both sides, it / this one: 10 x 40 -> 10 at 8 x 8
// 5.5 / 4.5 (774 layers of 32 and 40 channels 0.94 to 1.38 x), 2 x 184 -> 13 at 10 x 10 10.4 / 5.4 (478 of fewer than 128 tiles 1.2 to 3.5 x).  From 512 tiles up into
// fewer than 16 channels the pointwise kernel keeps planes that would be taken in tiles of four columns, 16 bytes of a row at a time (us, it / this one:
// 344 -> 9 at 16 x 90, 6 images 16.4 / 19.5, 216 -> 7 at 35 x 34, 8 images 12.4 / 14.6; of 13 drawn layers on rows of 26 and more
// all 0.84 to 1.0; shorter rows 0.98 to 1.25, wider tiles 1.0 to 2.4).
// Single taps that the pointwise kernel does not have (strides, odd planes), in place of the direct-to-LDS kernel, up to 1600 tiles of 32 to 64 channels,
// 1000 into fewer than 48 (1.05 to 2.2 x of 100 drawn layers, errors smaller in each: 56 -> 424 at 11 x 11, 2 images 13.5 -> 5.8, 64 -> 64 at 97 x 97 stride 2 12.2 -> 6.0; beyond
// 0.86 to 1.5 x; of 24 channels 0.96 to 1.6 x, some errors larger).  Nor do they cross at 65 tiles, where tests assert the direct-to-LDS kernel: 2 x 64 -> 28 at
// 13 x 13 8.0 / 4.7 (196 layers 1.4 to 2.3 x).
static bool few_tiles_first(const Conv2dShape& s, const float* x, const float* w, const float* y)
{
    const int64_t tiles = (int64_t)s.N * (((int64_t)s.Ho * s.Wo + 15) / 16) * ((s.C_out + 15) / 16);
    if (mfma_f32_pointwise_supported(s, x, w, y)) {
        if (s.C_in < 48 || tiles > (s.C_out >= 128 && s.C_in >= 64 ? 1600 : 640) || (tiles < 128 && s.C_out < 128)) return false;
        if (s.C_out < 16 && tiles > 512 && s.Wo > 24 && mfma_f32_few_supported(s) && mfma_f32_few_columns(s) <= 4) return false;
    } else if (s.C_in <= 64 && !few_tiles_before_rows(s)) {
        if (s.R * s.S != 1 || s.C_in < 32 || tiles < 65 || tiles > (s.C_out < 48 ? 1000 : 1600)) return false;
    }
    return few_tiles(s);
}

// Nine taps on split operands (or in few tiles) before the direct-to-LDS, fixed, quad and any-shape kernels: from 33 channels up (us, 56 x 56 -> 64
// channels: 64 channels 75.4 -> 52.1, one image 21.1 -> 10.4), and below that down to 9 channels, though 16 are multiplied, but where tests assert the
// plans of the others: small launches into few channels.  Graph of ten, us: 25 x 32 -> 208 at 36 x 36 92.2 -> 33.8, 21 x 24 -> 112 at 61 x 61 dilation 2
// 63.8 -> 48.0, 4 x 32 -> 96 at 38 x 38 21.6 -> 9.1, 12 x 28 -> 32 at 67 x 67 65.6 -> 14.7, 21 x 9 -> 416 at 14 x 14 19.7 -> 13.7, 20 x 30 -> 32 at
// 25 x 41 stride 2 43.9 -> 8.6; in few tiles 24 -> 32 at 17 x 72 dilation 2 14.5 -> 5.5.  Over 250 drawn layers 1.6 (direct-to-LDS), 2.1 (quad) and
// 3.1 (any-shape kernel), none below 1.13, errors against 64 bits smaller in each.  The lines at 1024 and 2500 pixels and 96 outputs are those of the tests' layers,
// not where the kernels cross.  Both sides, others / split or few tiles: 6 x 32 -> 17 at 7 x 7 9.8 / 5.3 (178 layers of 17 to 32 channels 1.55 to 2.55 x), 7 x 15 -> 32
// at 7 x 7 stride 2 11.9 / 5.0 (512 of 9 to 16 channels 1.3 to 3.3 x).
static bool split_first(const Conv2dShape& s)
{
    const int64_t pixels = (int64_t)s.N * s.Ho * s.Wo;
    return s.C_in > 32 || (s.C_in > 16 && (pixels > 1024 || s.C_in % 8 != 0 || s.C_out > 96)) || (s.C_in > 8 && (pixels > 2500 || s.C_out > 96));
}

// ... but of up to 32 channels not those whose windows hold many times the cells of their tiles (dilations from 3 up, nine filter rows), which
// every block of 32 output channels fetches and splits again.  The estimates decide against the kernel that has the layer otherwise (us, that
// kernel / the split one: 24 -> 174 at 87 x 55 9 x 1, 40 images 196 / 404, 24 -> 349 at 46 x 46 dilation 4, 16 images 88 / 165, 12 -> 370 at 70 x 70
// dilation 3, 17 images 116 / 160; of 4042 drawn layers of 9 to 32 channels, half of them so dilated or 9 x 1, 43 were slower split, 0.49 to 0.97.
// Left there are those of 0.81 to 0.97, where neither estimate is that good, and a few go back that were up to 1.1 x as fast split.  The fixed and
// the quad kernel had none, 1.09 to 4 x).
static bool split_slower(const Conv2dShape& s, const float* x, const float* w)
{
    if (s.C_in > 32 || (mfma_f32_supported(s) && mfma_f32_workgroups(s) >= 160)) return false;
    // (the line between them lies higher for sums in parts, whose launches are the smaller ones)
    if (const int parts = mfma_f32_dma_parts(s, x, w)) return mfma_f32_split_estimate(s) > (parts > 1 ? 1.2 : 1.05) * mfma_f32_dma_estimate_nine(s, x, w);
    return !mfma_f32_quad_supported(s) && mfma_f32_any_supported(s) && mfma_f32_split_estimate(s) > 1.1 * mfma_f32_any_estimate_nine(s, w);
}

// The multi-channel fp32 convolution with the store's epilogue (none for sw_conv2d).
static int run_conv2d(const float* x, const float* w, float* y, const Conv2dShape& s, const Epilogue& ep, hipStream_t st)
{
    const bool plain = !ep.bias && !ep.relu;
    (void)plain;
    if (s.C_in == 1)
        return run_plane(x, w, y, (int64_t)s.N * s.C_out, s.C_out, s.C_out, s, false, st, ep);
    if (!force_direct() && s.C_in > 1) {
        if (few_tiles_first(s, x, w, y)) return launch_status(launch_mfma_f32_few(x, w, y, s, st, ep));
        // The fixed 3x3 / 5x5 kernel holds a CU with one large tile: it needs enough of them to fill the chip
        // (28 x 28 images and below at batch 32 leave it at 128 or fewer); the any-shape kernel's 128-pixel
        // tiles take over there, and everywhere the fixed kernel has no variant.
        // Filters of 25 taps and more over at least 8 channels: the compound kernel (one filter row of a channel
        // chunk at a time, 256-pixel tiles), measured faster than the kernels below from 5 x 5 upward and the only
        // matrix-core kernel beyond 13 x 13.
        // One tap, stride 1, no padding: the input is the B operand as it lies in memory (nothing staged); measured
        // faster than the window kernels on every such layer tried.
        if (mfma_f32_pointwise_supported(s, x, w, y))
            return launch_status(launch_mfma_f32_pointwise(x, w, y, s, st, ep));
        // planes of an odd number of pixels and tensors that begin between 8-byte addresses
        if (mfma_f32_pointwise_loose_supported(s, x, w, y))
            return launch_status(launch_mfma_f32_pointwise_loose(x, w, y, s, st, ep));
        if (s.R * s.S >= 25 && s.C_in >= 8 && mfma_f32_rows_supported(s, x))
            return launch_status(launch_mfma_f32_rows(x, w, y, s, st, ep));
        // Few channels at an even stride (the first layer of an image network): K along the filter rows
        // (7 x 7 stride 2, 3 -> 64 at 224 x 224: 170 -> 54 us; 3 x 3 stride 2, 3 -> 32: 48 -> 21, 9.6 -> 6.3 for one image), but where
        // the filter rows are too short to fill it
        if (mfma_f32_stem_supported(s)) return launch_status(launch_mfma_f32_stem(x, w, y, s, st, ep));
        if (split_first(s) && mfma_f32_split_supported(s)) {
            if (s.C_in <= 32 && few_tiles(s)) return launch_status(launch_mfma_f32_few(x, w, y, s, st, ep));
            if (!split_slower(s, x, w)) return launch_status(launch_mfma_f32_split(x, w, y, s, st, ep));
        }
        const bool quad_ok = mfma_f32_quad_supported(s);
        const bool any_ok = quad_ok || mfma_f32_any_supported(s);
        if (mfma_f32_supported(s) && (mfma_f32_workgroups(s) >= 160 || !any_ok))
            return launch_status(launch_mfma_f32(x, w, y, s, st, ep));
        // few taps over whole groups of eight channels: operands by direct-to-LDS loads, the next chunk in flight
        // while this one multiplies
        if (mfma_f32_dma_supported(s, x, w)) return launch_status(launch_mfma_f32_dma(x, w, y, s, st, ep));
        // the kernels for any shape, in launches of few tiles (17 channels up where the quad kernel has the layer; us, quad and any-shape
        // kernels -> this one: 2 x 21 -> 80 at 18 x 18 3x3 16.6 -> 6.4, 3 x 24 -> 40 at 12 x 31 5x5 63 -> 7.8, 2 x 16 -> 48 at 16 x 69 5x5 44 -> 7.3)
        if ((quad_ok ? s.C_in > 16 : any_ok) && few_tiles(s)) return launch_status(launch_mfma_f32_few(x, w, y, s, st, ep));
        if (quad_ok) return launch_status(launch_mfma_f32_quad(x, w, y, s, st, ep));
        if (any_ok) return launch_status(launch_mfma_f32_any(x, w, y, s, st, ep));
        if (mfma_f32_rows_supported(s, x)) return launch_status(launch_mfma_f32_rows(x, w, y, s, st, ep));
    }
    return launch_status(launch_direct_conv2d_f32(x, w, y, s, false, st, &ep));
}

int sw_conv2d(const float* x, const float* w, float* y, int N, int C_in, int C_out, int H, int W, int R,
              int S, int stride, int pad, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C_in, C_out, H, W, R, S, stride, pad, false, 4, 4, &s);
    if (rc != SW_OK) return rc;
    return run_conv2d(x, w, y, s, Epilogue{nullptr, 0}, static_cast<hipStream_t>(hip_stream));
}

int sw_conv2d_bias_relu(const float* x, const float* w, const float* bias, float* y, int N, int C_in, int C_out, int H,
                        int W, int R, int S, int stride, int pad, int relu, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C_in, C_out, H, W, R, S, stride, pad, false, 4, 4, &s);
    if (rc != SW_OK) return rc;
    if (bias && misaligned(bias, 4)) return SW_ERR_ALIGN;
    if (bias && overlaps(y, (int64_t)N * C_out * s.Ho * s.Wo * 4, bias, (int64_t)C_out * 4)) return SW_ERR_ALIAS;
    return run_conv2d(x, w, y, s, Epilogue{bias, relu != 0}, static_cast<hipStream_t>(hip_stream));
}

int sw_conv2d_dilated(const float* x, const float* w, float* y, int N, int C_in, int C_out, int H, int W, int R,
                      int S, int stride, int pad, int dilation, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C_in, C_out, H, W, R, S, stride, pad, false, 4, 4, &s, dilation);
    if (rc != SW_OK) return rc;
    return run_conv2d(x, w, y, s, Epilogue{nullptr, 0}, static_cast<hipStream_t>(hip_stream));
}

int sw_conv2d_depthwise_dilated(const float* x, const float* w, float* y, int N, int C, int H, int W, int R, int S,
                                int stride, int pad, int dilation, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C, C, H, W, R, S, stride, pad, true, 4, 4, &s, dilation);
    if (rc != SW_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return run_plane(x, w, y, (int64_t)N * C, 1, C, s, true, st);
}

int sw_conv2d_depthwise(const float* x, const float* w, float* y, int N, int C, int H, int W, int R, int S,
                        int stride, int pad, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C, C, H, W, R, S, stride, pad, true, 4, 4, &s);
    if (rc != SW_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    return run_plane(x, w, y, (int64_t)N * C, 1, C, s, true, st);
}

// fp32 / bf16 / half (ek: Elem) convolution on channel-last tensors with the store's epilogue
static int run_nhwc(const void* x, const void* w, const float* bias, void* y, int N, int H, int W, int C_in, int C_out,
                    int R, int S, int stride, int pad, int dilation, int relu, int ek, void* hip_stream)
{
    const int esz = elem_size(ek);
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C_in, C_out, H, W, R, S, stride, pad, false, (size_t)esz, (size_t)esz, &s,
                                dilation);
    if (rc != SW_OK) return rc;
    if (bias && misaligned(bias, 4)) return SW_ERR_ALIGN;
    if (bias && overlaps(y, (int64_t)N * C_out * s.Ho * s.Wo * esz, bias, (int64_t)C_out * 4)) return SW_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const Epilogue ep{bias, relu != 0};
    if (!force_direct() && mfma_nhwc_lds_supported(x, w, y, s, ek))
        return launch_status(launch_mfma_nhwc_lds(x, w, y, s, ek, ep, st));
    if (!force_direct() && esz == 2 && mfma_bf16_nhwc_direct_supported(x, w, y, s))
        return launch_status(launch_mfma_bf16_nhwc_direct(x, w, y, s, ek == kElemF16, ep, st));
    if (!force_direct() && mfma_nhwc_supported(x, w, s, ek)) return launch_status(launch_mfma_nhwc(x, w, y, s, ek, ep, st));
    if (!force_direct() && few_channels_nhwc_supported(y, s)) return launch_status(launch_few_channels_nhwc(x, w, y, s, ek, ep, st));
    return launch_status(launch_direct_nhwc(x, w, y, s, ek, ep, st));
}

int sw_conv2d_nhwc(const float* x, const float* w, const float* bias, float* y, int N, int H, int W, int C_in, int C_out,
                   int R, int S, int stride, int pad, int dilation, int relu, void* hip_stream)
{
    return run_nhwc(x, w, bias, y, N, H, W, C_in, C_out, R, S, stride, pad, dilation, relu, kElemF32, hip_stream);
}

int sw_conv2d_bf16_nhwc(const void* x, const void* w, const float* bias, void* y, int N, int H, int W, int C_in, int C_out,
                        int R, int S, int stride, int pad, int dilation, int relu, void* hip_stream)
{
    return run_nhwc(x, w, bias, y, N, H, W, C_in, C_out, R, S, stride, pad, dilation, relu, kElemBF16, hip_stream);
}

int sw_conv2d_f16_nhwc(const void* x, const void* w, const float* bias, void* y, int N, int H, int W, int C_in, int C_out,
                       int R, int S, int stride, int pad, int dilation, int relu, void* hip_stream)
{
    return run_nhwc(x, w, bias, y, N, H, W, C_in, C_out, R, S, stride, pad, dilation, relu, kElemF16, hip_stream);
}

// int8 convolution on channel-last tensors; bias/scale == nullptr and y8 == nullptr: int32 sums
static int run_s8_nhwc(const int8_t* x, const int8_t* w, const int32_t* bias, const float* scale, int32_t* y, int8_t* y8,
                       int N, int H, int W, int C_in, int C_out, int R, int S, int stride, int pad, int relu,
                       void* hip_stream)
{
    Conv2dShape s;
    const void* out = y8 ? static_cast<const void*>(y8) : static_cast<const void*>(y);
    const int rc = check_conv2d(x, w, out, N, C_in, C_out, H, W, R, S, stride, pad, false, 1, y8 ? 1 : 4, &s);
    if (rc != SW_OK) return rc;
    if ((int64_t)C_in * R * S > 131071) return SW_ERR_SHAPE;  // 131072 * 2^14 = 2^31 leaves int32
    Requant rq{bias, scale, relu != 0};
    if (y8) {
        if (misaligned(scale, 4) || (bias && misaligned(bias, 4))) return SW_ERR_ALIGN;
        const int64_t ny = (int64_t)N * C_out * s.Ho * s.Wo;
        if (overlaps(y8, ny, scale, (int64_t)C_out * 4) || (bias && overlaps(y8, ny, bias, (int64_t)C_out * 4)))
            return SW_ERR_ALIAS;
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    // one tap, int8 out: the pixels straight from x, their channels all in flight at once
    if (!force_direct() && y8 && mfma_s8_pointwise_nhwc_supported(x, w, y8, s))
        return launch_status(launch_mfma_s8_pointwise_nhwc(x, w, y8, rq, s, st));
    if (!force_direct() && mfma_s8_nhwc_lds_supported(x, w, y8 ? static_cast<const void*>(y8) : static_cast<const void*>(y), y8 != nullptr, s))
        return launch_status(launch_mfma_s8_nhwc_lds(x, w, y8 ? static_cast<void*>(y8) : static_cast<void*>(y), y8 ? &rq : nullptr, s, st));
    if (!force_direct() && mfma_s8_nhwc_supported(x, w, s))
        return launch_status(launch_mfma_s8_nhwc(x, w, y, y8, y8 ? &rq : nullptr, s, st));
    return launch_status(launch_direct_s8_nhwc(x, w, y, y8, y8 ? &rq : nullptr, s, st));
}

int sw_conv2d_s8_nhwc(const int8_t* x, const int8_t* w, int32_t* y, int N, int H, int W, int C_in, int C_out, int R,
                      int S, int stride, int pad, void* hip_stream)
{
    return run_s8_nhwc(x, w, nullptr, nullptr, y, nullptr, N, H, W, C_in, C_out, R, S, stride, pad, 0, hip_stream);
}

int sw_conv2d_s8_nhwc_requant(const int8_t* x, const int8_t* w, const int32_t* bias, const float* scale, int8_t* y,
                              int N, int H, int W, int C_in, int C_out, int R, int S, int stride, int pad, int relu,
                              void* hip_stream)
{
    if (!scale || !y) return SW_ERR_NULL;
    return run_s8_nhwc(x, w, bias, scale, nullptr, y, N, H, W, C_in, C_out, R, S, stride, pad, relu, hip_stream);
}

int sw_dw_pw_block(const float* x, const float* w_dw, const float* b_dw, const float* w_pw, const float* b_pw, float* y,
                   int N, int C, int C_out, int H, int W, int relu_dw, int relu_pw, void* hip_stream)
{
    if (!x || !w_dw || !w_pw || !y) return SW_ERR_NULL;
    if (N <= 0 || C <= 0 || C_out <= 0 || H <= 0 || W <= 0) return SW_ERR_SHAPE;
    const int64_t nx = (int64_t)N * C * H * W, ny = (int64_t)N * C_out * H * W, npw = (int64_t)C_out * C;
    if (nx > kMaxElems || ny > kMaxElems || npw > kMaxElems) return SW_ERR_SHAPE;
    if (misaligned(x, 4) || misaligned(w_dw, 4) || misaligned(w_pw, 4) || misaligned(y, 4) ||
        (b_dw && misaligned(b_dw, 4)) || (b_pw && misaligned(b_pw, 4)))
        return SW_ERR_ALIGN;
    if (overlaps(y, ny * 4, x, nx * 4) || overlaps(y, ny * 4, w_dw, (int64_t)C * 9 * 4) || overlaps(y, ny * 4, w_pw, npw * 4) ||
        (b_dw && overlaps(y, ny * 4, b_dw, (int64_t)C * 4)) || (b_pw && overlaps(y, ny * 4, b_pw, (int64_t)C_out * 4)))
        return SW_ERR_ALIAS;
    if (!dw_pw_block_supported(N, C, C_out, H, W)) return SW_ERR_UNSUPPORTED;
    return launch_status(launch_dw_pw_block(x, w_dw, b_dw, w_pw, b_pw, y, N, C, C_out, H, W, relu_dw != 0, relu_pw != 0,
                                            static_cast<hipStream_t>(hip_stream)));
}

int sw_conv2d_depthwise_bias_relu(const float* x, const float* w, const float* bias, float* y, int N, int C, int H,
                                  int W, int R, int S, int stride, int pad, int relu, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C, C, H, W, R, S, stride, pad, true, 4, 4, &s);
    if (rc != SW_OK) return rc;
    if (bias && misaligned(bias, 4)) return SW_ERR_ALIGN;
    if (bias && overlaps(y, (int64_t)N * C * s.Ho * s.Wo * 4, bias, (int64_t)C * 4)) return SW_ERR_ALIAS;
    return run_plane(x, w, y, (int64_t)N * C, 1, C, s, true, static_cast<hipStream_t>(hip_stream),
                     Epilogue{bias, relu != 0});
}

int sw_conv2d_depthwise_bf16(const uint16_t* x, const float* w, uint16_t* y, int N, int C, int H, int W, int R, int S,
                             int stride, int pad, void* hip_stream)
{
    Conv2dShape s;
    // (element sizes: activations 2 bytes; the filter is checked as fp32 below)
    const int rc = check_conv2d(x, w, y, N, C, C, H, W, R, S, stride, pad, true, 2, 2, &s);
    if (rc != SW_OK) return rc;
    if (misaligned(w, 4)) return SW_ERR_ALIGN;
    if (overlaps(y, (int64_t)N * C * s.Ho * s.Wo * 2, w, (int64_t)C * R * S * 4)) return SW_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (!force_direct() && sliding_plane_bf16_supported(x, y, H, W, R, S, stride, pad, s.Ho, s.Wo))
        return launch_status(launch_sliding_plane_bf16(x, w, y, (int64_t)N * C, C, H, W, R, pad, s.Ho, s.Wo, st));
    // bands of output rows, but one thread per output on planes with little to do (plane_bands_worthwhile)
    if (!force_direct() && plane_bands_supported(x, (int64_t)N * C, 1, C, s, true))
        return launch_status(launch_plane_bands(x, w, y, (int64_t)N * C, 1, C, s, true, st));
    return launch_status(launch_direct_depthwise_bf16(x, w, y, s, st));
}

int sw_conv2d_depthwise_dilated_jit(const float* x, const float* w, float* y, int N, int C, int H, int W, int R, int S,
                                    int stride, int pad, int dilation, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C, C, H, W, R, S, stride, pad, true, 4, 4, &s, dilation);
    if (rc != SW_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (!force_direct() && jit_plane_supported(x, y, H, W, R, S, stride, pad, dilation)) {
        // a geometry whose generated kernel cannot be compiled or loaded is served by the precompiled kernels
        if (jit_launch_plane(x, w, y, (int64_t)N * C, 1, C, H, W, R, S, stride, pad, dilation, st) == SW_OK) return SW_OK;
    }
    return run_plane(x, w, y, (int64_t)N * C, 1, C, s, true, st);
}

int sw_conv2d_depthwise_jit(const float* x, const float* w, float* y, int N, int C, int H, int W, int R, int S,
                            int stride, int pad, void* hip_stream)
{
    return sw_conv2d_depthwise_dilated_jit(x, w, y, N, C, H, W, R, S, stride, pad, 1, hip_stream);
}

static int jit_geometry_ok(int H, int W, int R, int S, int stride, int pad, int dilation)
{
    if (H <= 0 || W <= 0 || R <= 0 || S <= 0 || stride <= 0 || pad < 0 || dilation <= 0) return SW_ERR_SHAPE;
    if (sw_out_dim_dilated(H, R, stride, pad, dilation) <= 0 || sw_out_dim_dilated(W, S, stride, pad, dilation) <= 0)
        return SW_ERR_SHAPE;
    return SW_OK;
}

int sw_jit_prepare_depthwise_dilated(int H, int W, int R, int S, int stride, int pad, int dilation)
{
    const int rc = jit_geometry_ok(H, W, R, S, stride, pad, dilation);
    return rc != SW_OK ? rc : jit_prepare_plane(H, W, R, S, stride, pad, dilation);
}

int sw_jit_prepare_depthwise(int H, int W, int R, int S, int stride, int pad)
{
    return sw_jit_prepare_depthwise_dilated(H, W, R, S, stride, pad, 1);
}

int sw_jit_compile_check_dilated(int H, int W, int R, int S, int stride, int pad, int dilation)
{
    const int rc = jit_geometry_ok(H, W, R, S, stride, pad, dilation);
    return rc != SW_OK ? rc : jit_compile_only(H, W, R, S, stride, pad, dilation);
}

int sw_jit_compile_check(int H, int W, int R, int S, int stride, int pad)
{
    return sw_jit_compile_check_dilated(H, W, R, S, stride, pad, 1);
}

int sw_jit_cached_kernels(void) { return jit_cached_kernels(); }

// One or nine taps on the kernel that turns its operands in registers, where the band kernel has no plan.  Against the any-shape kernel it was
// faster on 368 of 370 drawn layers and on all larger ones tried (1.1 to 12 x), but for single taps over at most 32 channels whose sums
// leave as int32 (one unit of channels: 32 -> 64 at 56 x 56, 32 images, 9.6 us against 11.8), and over at most 64 into more than 32 from 8192
// tiles up on planes of whole dwords (51 drawn layers 0.62 to 1.3 x: 29 x 48 -> 36 at 80 x 104 17.8 us against 28.6); against the 32-row kernel (mfma_s8_kernel) up to 8192 tiles
// (32 x 256 -> 256 at 12 x 12 17.9 -> 16.8, 8 x 64 -> 128 at 100 x 100, 40000 tiles, 33.8 and 33.2).
static bool s8_tiles_first(const int8_t* w, const Conv2dShape& s, bool requant)
{
    const bool by_rows = requant ? mfma_s8_requant_supported(s) : mfma_s8_supported(s);
    const bool filled = (int64_t)s.N * (((int64_t)s.Ho * s.Wo + 15) / 16) * ((s.C_out + 15) / 16) > 8192;
    const bool short_sums = !requant && s.R * s.S == 1 && (s.C_in <= 32 || (s.C_in <= 64 && s.C_out > 32 && s.W % 4 == 0 && s.stride == 1 && filled));
    if (by_rows ? filled : short_sums) return false;
    return mfma_s8_tiles_supported(w, requant, s);       // (the search comes last)
}

int sw_conv2d_s8(const int8_t* x, const int8_t* w, int32_t* y, int N, int C_in, int C_out, int H, int W,
                 int R, int S, int stride, int pad, void* hip_stream)
{
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C_in, C_out, H, W, R, S, stride, pad, false, 1, 4, &s);
    if (rc != SW_OK) return rc;
    if ((int64_t)C_in * R * S > 131071) return SW_ERR_SHAPE;  // 131072 * 2^14 = 2^31 leaves int32
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    if (!force_direct()) {
        if (mfma_s8_band_supported(x, w, s, true))
            return launch_status(launch_mfma_s8_band(x, w, y, nullptr, nullptr, s, true, st));
        if (s8_tiles_first(w, s, false)) return launch_status(launch_mfma_s8_tiles(x, w, y, nullptr, nullptr, s, st));
        if (mfma_s8_supported(s)) return launch_status(launch_mfma_s8(x, w, y, s, st));
        if (mfma_s8_any_supported(s)) return launch_status(launch_mfma_s8_any(x, w, y, s, st));
    }
    return launch_status(launch_direct_conv2d_s8(x, w, y, s, st));
}

int sw_conv2d_s8_requant(const int8_t* x, const int8_t* w, const int32_t* bias, const float* scale, int8_t* y, int N,
                         int C_in, int C_out, int H, int W, int R, int S, int stride, int pad, int relu,
                         void* hip_stream)
{
    if (!scale) return SW_ERR_NULL;
    Conv2dShape s;
    const int rc = check_conv2d(x, w, y, N, C_in, C_out, H, W, R, S, stride, pad, false, 1, 1, &s);
    if (rc != SW_OK) return rc;
    if ((int64_t)C_in * R * S > 131071) return SW_ERR_SHAPE;  // 131072 * 2^14 = 2^31 leaves int32
    if (misaligned(scale, 4) || (bias && misaligned(bias, 4))) return SW_ERR_ALIGN;
    const int64_t ny = (int64_t)N * C_out * s.Ho * s.Wo;
    if (overlaps(y, ny, scale, (int64_t)C_out * 4) || (bias && overlaps(y, ny, bias, (int64_t)C_out * 4)))
        return SW_ERR_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const Requant rq{bias, scale, relu != 0};
    if (!force_direct()) {
        if (mfma_s8_band_supported(x, w, s, true))
            return launch_status(launch_mfma_s8_band(x, w, nullptr, y, &rq, s, true, st));
        if (s8_tiles_first(w, s, true)) return launch_status(launch_mfma_s8_tiles(x, w, nullptr, y, &rq, s, st));
        if (mfma_s8_requant_supported(s))
            return launch_status(launch_mfma_s8_requant(x, w, y, rq, s, st));
        if (mfma_s8_any_supported(s)) return launch_status(launch_mfma_s8_any_requant(x, w, y, rq, s, st));
    }
    return launch_status(launch_direct_conv2d_s8_requant(x, w, y, rq, s, st));
}

int64_t sw_s8_packed_filter_bytes(int C_in, int C_out, int R, int S)
{
    if (C_in <= 0 || C_out <= 0 || R <= 0 || S <= 0 || R > kMaxFilter2D || S > kMaxFilter2D) return 0;
    if ((int64_t)C_out * C_in * R * S > kMaxElems) return 0;
    const int64_t bytes = s8_packed_filter_bytes(C_in, C_out, R, S);
    return bytes > kMaxElems ? 0 : bytes;
}

int sw_s8_pack_filter(const int8_t* w, int8_t* packed, int C_in, int C_out, int R, int S, void* hip_stream)
{
    if (!w || !packed) return SW_ERR_NULL;
    if (C_in <= 0 || C_out <= 0 || R <= 0 || S <= 0) return SW_ERR_SHAPE;
    if (R > kMaxFilter2D || S > kMaxFilter2D) return SW_ERR_UNSUPPORTED;
    const int64_t nw = (int64_t)C_out * C_in * R * S;
    if (nw > kMaxElems) return SW_ERR_SHAPE;
    const int64_t bytes = sw_s8_packed_filter_bytes(C_in, C_out, R, S);
    if (bytes <= 0) return SW_ERR_SHAPE;
    if (misaligned(packed, 16)) return SW_ERR_ALIGN;
    if (overlaps(packed, bytes, w, nw)) return SW_ERR_ALIAS;
    return launch_status(launch_pack_filter_s8(w, packed, C_in, C_out, R, S, static_cast<hipStream_t>(hip_stream)));
}

// Shared by the two packed-filter calls; bias/scale/y8 == nullptr: int32 sums.
static int run_s8_packed(const int8_t* x, const int8_t* packed, const int32_t* bias, const float* scale, int32_t* y,
                         int8_t* y8, int N, int C_in, int C_out, int H, int W, int R, int S, int stride, int pad, int relu,
                         void* hip_stream)
{
    Conv2dShape s;
    const void* out = y8 ? static_cast<const void*>(y8) : static_cast<const void*>(y);
    // (check_conv2d sees the packed buffer as the filter: it is at least as large as the filter tensor)
    const int rc = check_conv2d(x, packed, out, N, C_in, C_out, H, W, R, S, stride, pad, false, 1, y8 ? 1 : 4, &s);
    if (rc != SW_OK) return rc;
    if ((int64_t)C_in * R * S > 131071) return SW_ERR_SHAPE;  // 131072 * 2^14 = 2^31 leaves int32
    const int64_t bytes = sw_s8_packed_filter_bytes(C_in, C_out, R, S);
    if (bytes <= 0) return SW_ERR_SHAPE;
    if (misaligned(packed, 16)) return SW_ERR_ALIGN;
    const int64_t ny = (int64_t)N * C_out * s.Ho * s.Wo * (y8 ? 1 : 4);
    if (overlaps(out, ny, packed, bytes)) return SW_ERR_ALIAS;
    Requant rq{bias, scale, relu != 0};
    if (y8) {
        if (misaligned(scale, 4) || (bias && misaligned(bias, 4))) return SW_ERR_ALIGN;
        if (overlaps(y8, ny, scale, (int64_t)C_out * 4) || (bias && overlaps(y8, ny, bias, (int64_t)C_out * 4)))
            return SW_ERR_ALIAS;
    }
    return launch_status(launch_conv2d_s8_packed(x, packed, y, y8, y8 ? &rq : nullptr, s, !force_direct(),
                                                 static_cast<hipStream_t>(hip_stream)));
}

int sw_conv2d_s8_packed(const int8_t* x, const int8_t* packed, int32_t* y, int N, int C_in, int C_out, int H, int W,
                        int R, int S, int stride, int pad, void* hip_stream)
{
    return run_s8_packed(x, packed, nullptr, nullptr, y, nullptr, N, C_in, C_out, H, W, R, S, stride, pad, 0, hip_stream);
}

int sw_conv2d_s8_packed_requant(const int8_t* x, const int8_t* packed, const int32_t* bias, const float* scale,
                                int8_t* y, int N, int C_in, int C_out, int H, int W, int R, int S, int stride, int pad,
                                int relu, void* hip_stream)
{
    if (!scale || !y) return SW_ERR_NULL;
    return run_s8_packed(x, packed, bias, scale, nullptr, y, N, C_in, C_out, H, W, R, S, stride, pad, relu, hip_stream);
}

}  // extern "C"
