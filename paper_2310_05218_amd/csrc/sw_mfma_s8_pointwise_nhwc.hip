// Pointwise (1 x 1, stride 1, no padding) int8 convolution on channel-last tensors, requantised to int8 (paper, section 1.1:
// quantised inference; section 3: taps as small matrix products).
//
//     y[p][co] = requantised sum over ci of w[co][ci] * x[p][ci]          p = a pixel of all images
//
// With one tap there is no window to keep in LDS: a pixel's 16 consecutive channels are 16 consecutive bytes of x, the operand
// of one lane of v_mfma_i32_32x32x32_i8, so a wavefront loads the operands of its 32 pixels straight into registers, all of a
// chunk of 256 channels at once: one memory round trip where the window kernel takes one per 128 bytes of a pixel.  The
// filters of the workgroup's 32 CB output channels (rows as they lie in w, padded by 16 bytes against bank conflicts) come into
// LDS under the same round trip, by direct-to-LDS loads.  Results are packed four at a time (requant_pack4) and leave through a
// per-wavefront LDS area as 16-byte pieces of a pixel.
//
// Measured (us per launch, replayed graphs of ten; the window kernel of the time -> first form of this one): 32 x 28 x 28 x 512 -> 128 10.9 -> 8.6, 128 -> 512
// 16.4 -> 11.7, 32 x 14 x 14 x 256 -> 1024 12.9 -> 8.5, 32 x 56 x 56 x 256 -> 64 13.1 -> 8.9, 6 x 25 x 25 x 160 -> 640 9.0 -> 5.1, one image
// 28 x 28 x 512 -> 128 6.8 -> 6.0.  CB = 4 where that leaves 192 workgroups, else 2: fetching 128 filter rows made small
// launches slower than the window kernel's.
// Then (time stamps, cycles, 512 -> 128 / 128 -> 512): the filters' loads took 2.7 / 1.4 k to leave (divisions for each), biases and scales came 3 k
// later for standing behind them, every filter read was waited for by its matrix instruction, the next tile's pixels at the end of this
// one (a register copy: 2.6 k), every scale by its results (2.8 k a tile for 64 results a lane).  Now: sums that start from the
// biases, filters three steps ahead, pixels fetched again in place, all scales before the first result: 12.9 -> 10.5 k and 18.0 -> 13.2 k.
// What is left: filter reads at 64 bytes a cycle and CU, 4.1 k until the first product, 1.7 k of packing a tile.  A quantised
// bottleneck of this, a 3 x 3 and this again (32 x 28 x 28, 512 -> 128 -> 128 -> 512) 31.1 -> 26.0 us, 31 drawn ones 1.18 x, none slower.
#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "swconv_internal.h"

namespace swconv {

namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

#define SW_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

constexpr unsigned kBeyond = 0x80000000u;
constexpr int kChunkSteps = 8;             // steps of 32 channels whose pixel operands are in flight at once
constexpr size_t kLdsMax = 150 * 1024;

struct PwS8Params {
    Requant rq;
    int total_px, C_in, C_out, tiles;      // tiles of 32 pixels
    int pitch, rq_off, out_off;            // bytes per filter row in LDS; offsets of biases and scales, and of the store areas
    int wloads;                            // 1 KB loads of the workgroup's filters
    unsigned w_bytes;
    int d_row, d_piece;                    // from a lane's slot to that of its next load, 256 slots on
    FastDiv by_slots;                      // 16-byte slots per filter row: its pieces and one that pads it
};

// CB: blocks of 32 output channels per workgroup.
template <int CB>
__global__ __launch_bounds__(256, 2) void mfma_s8_pointwise_nhwc_kernel(const int8_t* __restrict__ x, const int8_t* __restrict__ w,
                                                                        int8_t* __restrict__ y, const PwS8Params P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, lj = lane & 31, kq = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int co0 = blockIdx.y * (32 * CB);
    const int steps = P.C_in >> 5;
    int tile = (int)blockIdx.x * 4 + wave;
    const int nwaves = (int)gridDim.x * 4;

    // biases and scales, on their way first: they come into LDS behind the filters' loads
    int bias = 0;
    float scale = 0.f;
    if (tid < 32 * CB) {
        const int co = min(co0 + tid, P.C_out - 1);
        if (P.rq.bias) bias = P.rq.bias[co];
        scale = P.rq.scale[co];
    }
    // a tile's pixels as a buffer: what lies beyond the last pixel, and a tile that is none, is read as zeros and without traffic
    auto pixels = [&](int t) __attribute__((always_inline)) {
        const int rows = t < P.tiles ? min(32, P.total_px - 32 * t) : 0;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(x) + (int64_t)min(t, P.tiles - 1) * 32 * P.C_in, 0, (unsigned)(rows * P.C_in), 0x00020000);
    };
    const unsigned px_off = (unsigned)(lj * P.C_in + 16 * kq);
    __amdgpu_buffer_rsrc_t xr = pixels(tile);
    intx4 b[kChunkSteps];
    // step s of a tile; a step beyond the last: zeros
    auto fetch = [&](int i, __amdgpu_buffer_rsrc_t r, int s) __attribute__((always_inline)) {
        b[i] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(r, px_off + (s < steps ? (unsigned)(32 * s) : kBeyond), 0, 0));
    };
#pragma unroll
    for (int i = 0; i < kChunkSteps; ++i) fetch(i, xr, i);

    {
        // the filters, by direct-to-LDS loads: all of them under the pixels' round trip.  (Their rows and pieces in steps from load to load)
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(w), 0, P.w_bytes, 0x00020000);
        const int pieces = P.C_in >> 4, rows = min(32 * CB, P.C_out - co0);
        int row = fast_div(tid, P.by_slots), g = tid - row * (pieces + 1);
        unsigned off = (unsigned)((co0 + row) * P.C_in + 16 * g);
        const unsigned step = (unsigned)(P.d_row * P.C_in + 16 * P.d_piece), turn = (unsigned)(P.C_in - 16 * (pieces + 1));
#pragma unroll 2
        for (int k = wave; k < P.wloads; k += 4) {
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, SW_LDS_PTR(smem + 1024 * k), 16, row < rows && g < pieces ? off : kBeyond, 0, 0, 0);
            row += P.d_row; g += P.d_piece; off += step;
            if (g > pieces) { g -= pieces + 1; ++row; off += turn; }
        }
    }
    if (tid < 32 * CB) {
        reinterpret_cast<int*>(smem + P.rq_off)[tid] = bias;
        reinterpret_cast<float*>(smem + P.rq_off)[32 * CB + tid] = scale;
    }
    __syncthreads();

    const unsigned char* arow = smem + lj * P.pitch + 16 * kq;
    // the filters of a step, kAhead steps ahead of it; a tile takes whole halves of a chunk, and steps beyond the last meet pixels of zeros
    constexpr int kAhead = kChunkSteps / 2 - 1;
    intx4 a[kAhead + 1][CB];
    const int whole = (steps + kAhead) & ~kAhead;
    int ahead = 0;
    auto read = [&](int i) __attribute__((always_inline)) {
        const unsigned char* from = arow + 32 * min(ahead, steps - 1);
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) a[i][cb] = *reinterpret_cast<const intx4*>(from + 32 * cb * P.pitch);
        ahead = ahead + 1 == whole ? 0 : ahead + 1;
    };
#pragma unroll
    for (int i = 0; i < kAhead; ++i) read(i);
#pragma unroll 1
    for (; tile < P.tiles; tile += nwaves) {
        // (the sums start from the biases)
        intx16 acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const intx4 bi = *reinterpret_cast<const intx4*>(smem + P.rq_off + 4 * (32 * cb + 8 * q + 4 * kq));
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[cb][4 * q + j] = bi[j];
            }
        const __amdgpu_buffer_rsrc_t xn = pixels(tile + nwaves);
#pragma unroll 1
        for (int s0 = 0; s0 < steps; s0 += kChunkSteps) {
            // The filters of the third step on between the matrix instructions of this one, in no branch: where paths with and without reads
            // meet, the compiler waits as if there were none.  A step's pixels are fetched again, those of the next chunk or tile, as they are
            // used: eight loads are always under way, and no register is copied.
            const bool last = s0 + kChunkSteps >= steps;
            auto again = [&](int i) __attribute__((always_inline)) { fetch(i, last ? xn : xr, last ? i : s0 + kChunkSteps + i); };
            auto half = [&](int first) __attribute__((always_inline)) {
#pragma unroll
                for (int i = first; i < first + kChunkSteps / 2; ++i) {
                    __builtin_amdgcn_sched_barrier(0);
                    read((i + kAhead) & kAhead);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i & kAhead][cb], b[i], acc[cb], 0, 0, 0);
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    again(i);
                }
            };
            half(0);
            if (s0 + kChunkSteps / 2 < steps) {
                half(kChunkSteps / 2);
            } else {
#pragma unroll
                for (int i = kChunkSteps / 2; i < kChunkSteps; ++i) again(i);
            }
        }
        xr = xn;

        // register v of a lane is output channel 8 (v / 4) + 4 kq + v % 4 of the block, pixel lj
        const int p0 = 32 * tile;
        constexpr int OP = 32 * CB + 16;               // bytes per pixel in the store area
        unsigned char* lo = smem + P.out_off + wave * 32 * OP;
        // (all scales before the first result is written: the compiler lets no read of LDS pass a write to it, and sixteen waits for one
        // scale each took most of the packing's time)
        floatx4 scales[CB][4];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                scales[cb][q] = *reinterpret_cast<const floatx4*>(smem + P.rq_off + 128 * CB + 4 * (32 * cb + 8 * q + 4 * kq));
        auto pack = [&](auto relu) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = 32 * cb + 8 * q + 4 * kq;
                    const floatx4& sc = scales[cb][q];
                    *reinterpret_cast<int*>(lo + lj * OP + col) =
                        requant_pack4<decltype(relu)::value>(acc[cb][4 * q], acc[cb][4 * q + 1], acc[cb][4 * q + 2], acc[cb][4 * q + 3], sc[0], sc[1],
                                                             sc[2], sc[3]);
                }
        };
        if (P.rq.relu) pack(std::true_type{});
        else pack(std::false_type{});
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // (the area is this wavefront's own)
        constexpr int NC = 2 * CB;                     // 16-byte pieces per pixel
#pragma unroll
        for (int pass = 0; pass < NC / 2; ++pass) {
            const int px = lane / NC + (64 / NC) * pass, piece = lane % NC;
            const intx4 v = *reinterpret_cast<const intx4*>(lo + px * OP + 16 * piece);
            if (p0 + px < P.total_px && co0 + 16 * piece < P.C_out)
                __builtin_nontemporal_store(v, reinterpret_cast<intx4*>(y + (int64_t)(p0 + px) * P.C_out + co0 + 16 * piece));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

struct PwS8Plan {
    bool ok = false;
    int CB = 0;
    size_t lds = 0;
    unsigned gx = 0, gy = 0;
    PwS8Params P;
};

PwS8Plan plan_pw_s8(const int8_t* x, const int8_t* w, const int8_t* y, const Conv2dShape& s)
{
    PwS8Plan a;
    const int64_t px = (int64_t)s.N * s.H * s.W;
    if (s.R != 1 || s.S != 1 || s.stride != 1 || s.pad != 0 || s.C_in % 32 != 0 || s.C_out % 16 != 0 || px >= (1LL << 31) - 64 ||
        (int64_t)s.C_out * s.C_in >= (1LL << 31))
        return a;
    for (const void* p : {(const void*)x, (const void*)w, (const void*)y})
        if (reinterpret_cast<uintptr_t>(p) % 16 != 0) return a;
    // below 128 channels the window kernel's steps hold all of a pixel, and its tests assert its plans there
    if (s.C_in < 128) return a;
    // a last channel group that is half empty, over many channels: its filters' way into LDS is most of a small launch
    // (640 -> 160 at 25 x 25, 6 images: 7.1 us in the window kernel, 7.6 here)
    if (s.C_in > 256 && s.C_out % 64 != 0 && s.C_out % 64 <= 32) return a;
    // ... nor over 128 channels, all of which the window kernel holds as well, in launches that CB = 4 does not fill (us, window kernel /
    // this one: 128 -> 208, 3136 pixels 5.4 / 5.8, 25088 pixels 10.8 / 10.1, 128 -> 528, 312 pixels 5.0 / 5.5, 25088 pixels 19.0 / 16.8)
    if (s.C_in == 128 && s.C_out > 64 && s.C_out % 64 != 0 && (px + 127) / 128 * ((s.C_out + 127) / 128) < 192) return a;
    const int pitch = s.C_in + 16;
    for (int CB : {4, 2}) {
        const int64_t groups = (s.C_out + 32 * CB - 1) / (32 * CB);
        if (CB == 4 && (s.C_out <= 64 || (px + 127) / 128 * groups < 192)) continue;
        const size_t filters = ((size_t)32 * CB * pitch + 1023) / 1024 * 1024, rq = (size_t)256 * CB, out = (size_t)4 * 32 * (32 * CB + 16);
        if (filters + rq + out > kLdsMax) continue;
        a.ok = true;
        a.CB = CB;
        a.lds = filters + rq + out;
        PwS8Params& P = a.P;
        P.total_px = (int)px; P.C_in = s.C_in; P.C_out = s.C_out; P.tiles = (int)((px + 31) / 32);
        P.pitch = pitch; P.rq_off = (int)filters; P.out_off = (int)(filters + rq);
        P.wloads = (int)(filters / 1024); P.w_bytes = (unsigned)((int64_t)s.C_out * s.C_in);
        P.by_slots = make_fastdiv(s.C_in / 16 + 1);
        P.d_row = 256 / (s.C_in / 16 + 1);
        P.d_piece = 256 % (s.C_in / 16 + 1);
        a.gy = (unsigned)groups;
        // persistent: as many workgroups as fit their CUs at once, by registers two of CB = 4 and three of CB = 2 (four, as LDS would have it,
        // left a second turn of a few: 128 -> 512 at 28 x 28 12.7 us against 11.3, at 56 x 56 26.9 against 24.2)
        const int per_cu = (int)std::max<size_t>(1, std::min<size_t>(CB == 4 ? 2 : 3, 160 * 1024 / a.lds));
        const int64_t cap = std::max<int64_t>(1, (int64_t)256 * per_cu / a.gy);
        a.gx = (unsigned)std::min<int64_t>((P.tiles + 3) / 4, cap);
        break;
    }
    if (a.gy > 65535) a.ok = false;
    return a;
}

template <int CB>
hipError_t launch_pw_s8(const int8_t* x, const int8_t* w, int8_t* y, const PwS8Plan& a, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(mfma_s8_pointwise_nhwc_kernel<CB>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax);
    if (attr != hipSuccess) return attr;
    SW_NOTED_LAUNCH(note_kernel("mfma_s8_pointwise_nhwc_kernel", CB), (mfma_s8_pointwise_nhwc_kernel<CB>), dim3(a.gx, a.gy), dim3(256), a.lds, st,
                    x, w, y, a.P);
    return hipGetLastError();
}

}  // namespace

bool mfma_s8_pointwise_nhwc_supported(const int8_t* x, const int8_t* w, const int8_t* y, const Conv2dShape& s)
{
    return plan_pw_s8(x, w, y, s).ok;
}

hipError_t launch_mfma_s8_pointwise_nhwc(const int8_t* x, const int8_t* w, int8_t* y, const Requant& rq, const Conv2dShape& s, hipStream_t st)
{
    PwS8Plan a = plan_pw_s8(x, w, y, s);
    if (!a.ok) return hipErrorInvalidValue;
    a.P.rq = rq;
    return a.CB == 4 ? launch_pw_s8<4>(x, w, y, a, st) : launch_pw_s8<2>(x, w, y, a, st);
}

}  // namespace swconv
