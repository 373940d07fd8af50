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
// Measured (us per launch, replayed graphs of ten, window kernel -> this one): 32 x 28 x 28 x 512 -> 128 10.9 -> 8.6, 128 -> 512
// 16.4 -> 11.7, 32 x 14 x 14 x 256 -> 1024 12.9 -> 8.5, 32 x 56 x 56 x 256 -> 64 13.1 -> 8.9, 6 x 25 x 25 x 160 -> 640 9.0 -> 5.1, one image
// 28 x 28 x 512 -> 128 6.8 -> 6.0.  (With filters through registers in two round trips, ten instructions a packed result and more workgroups
// than run at once: 9.3, 14.0, 9.3, 10.3, 5.8, 6.3.)  CB = 4 where that leaves 192 workgroups, else 2: fetching 128 filter rows made small
// launches slower than the window kernel's.  Parts taken out of a copy (512 -> 128 / 128 -> 512): the pixels' loads 0.6 / 2.6, the
// filters' 0.8 / 1.0, packing 0.9 / 2.3, the stores 0.8 / 1.3; all chunks of 512 channels in flight at once was slower (10.2: registers).
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
    FastDiv by_slots;                      // 16-byte slots per filter row: its pieces and one that pads it
};

// CB: blocks of 32 output channels per workgroup.
template <int CB>
__global__ __launch_bounds__(256, 2) void mfma_s8_pointwise_nhwc_kernel(const int8_t* __restrict__ x, const int8_t* __restrict__ w,
                                                                        int8_t* __restrict__ y, const PwS8Params P)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lj = lane & 31, kq = lane >> 5;
    const int co0 = blockIdx.y * (32 * CB);
    const int steps = P.C_in >> 5;
    int tile = (int)blockIdx.x * 4 + wave;
    const int nwaves = (int)gridDim.x * 4;

    // (a pixel past the last one computes on the last and stores nothing)
    auto x_of = [&](int t) __attribute__((always_inline)) {
        const int p = min(32 * t + lj, P.total_px - 1);
        return x + (int64_t)p * P.C_in + 16 * kq;
    };
    intx4 b[kChunkSteps];
    auto fetch = [&](const int8_t* src, int s0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kChunkSteps; ++i) b[i] = *reinterpret_cast<const intx4*>(src + 32 * min(s0 + i, steps - 1));
    };
    const int8_t* xp = x_of(min(tile, P.tiles - 1));
    fetch(xp, 0);

    {
        // the filters, by direct-to-LDS loads: all of them under the pixels' round trip
        const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(const_cast<int8_t*>(w), 0, P.w_bytes, 0x00020000);
        const int pieces = P.C_in >> 4;
        const int wv = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll 2
        for (int k = wv; k < P.wloads; k += 4) {
            const int i = 64 * k + lane, row = fast_div(i, P.by_slots), g = i - row * (pieces + 1);
            const bool have = row < 32 * CB && g < pieces && co0 + row < P.C_out;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wr, SW_LDS_PTR(smem + 1024 * k), 16, have ? (unsigned)((co0 + row) * P.C_in + 16 * g) : kBeyond, 0, 0, 0);
        }
        if (tid < 32 * CB) {
            const int co = min(co0 + tid, P.C_out - 1);
            reinterpret_cast<int*>(smem + P.rq_off)[tid] = P.rq.bias ? P.rq.bias[co] : 0;
            reinterpret_cast<float*>(smem + P.rq_off)[32 * CB + tid] = P.rq.scale[co];
        }
    }
    __syncthreads();

    const unsigned char* arow = smem + lj * P.pitch + 16 * kq;
#pragma unroll 1
    for (; tile < P.tiles; tile += nwaves) {
        intx16 acc[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[cb][v] = 0;
        const bool more = tile + nwaves < P.tiles;
        const int8_t* xn = x_of(more ? tile + nwaves : tile);
#pragma unroll 1
        for (int s0 = 0; s0 < steps; s0 += kChunkSteps) {
            intx4 cur[kChunkSteps];
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) cur[i] = b[i];
            if (s0 + kChunkSteps < steps) fetch(xp, s0 + kChunkSteps);
            else if (more) fetch(xn, 0);
#pragma unroll
            for (int i = 0; i < kChunkSteps; ++i) {
                if (s0 + i >= steps) break;
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    const intx4 a = *reinterpret_cast<const intx4*>(arow + 32 * cb * P.pitch + 32 * (s0 + i));
                    acc[cb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, cur[i], acc[cb], 0, 0, 0);
                }
            }
        }
        xp = xn;

        // register v of a lane is output channel 8 (v / 4) + 4 kq + v % 4 of the block, pixel lj
        const int p0 = 32 * tile;
        constexpr int OP = 32 * CB + 16;               // bytes per pixel in the store area
        unsigned char* lo = smem + P.out_off + wave * 32 * OP;
        auto pack = [&](auto relu) __attribute__((always_inline)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = 32 * cb + 8 * q + 4 * kq;
                    const intx4 bi = *reinterpret_cast<const intx4*>(smem + P.rq_off + 4 * col);
                    const floatx4 sc = *reinterpret_cast<const floatx4*>(smem + P.rq_off + 128 * CB + 4 * col);
                    *reinterpret_cast<int*>(lo + lj * OP + col) =
                        requant_pack4<decltype(relu)::value>(acc[cb][4 * q] + bi[0], acc[cb][4 * q + 1] + bi[1], acc[cb][4 * q + 2] + bi[2],
                                                             acc[cb][4 * q + 3] + bi[3], sc[0], sc[1], sc[2], sc[3]);
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
