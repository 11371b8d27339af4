// Input transform V = B^T d B of eq. (2) (Barabasz & Gregg, arXiv 1905.05233)
// in registers: one thread per (tile, channel pair in 16-bit storage or one
// channel), the whole (m+2)^2 window in its registers.
//
// V[xi = a*alpha + b][tile][c] = sum_v (sum_u B^T[a][u] d[u][v]) B^T[b][v],
// d = the window whose top-left pixel is (ty*m - 1, tx*m - 1); pass 1 in
// ascending u and pass 2 in ascending v, fp32 fused multiply-adds from zero,
// rounded to the storage type at the store.
//
// What bounds it: alpha'^2 / m^2 times the input's bytes are written, so large
// layers run at the memory system's rate.  The threads of a workgroup take
// consecutive runs of V's planes (channels fastest), so every store of a wave is
// one contiguous piece and every window load covers consecutive NHWC channels;
// the overlap of neighbouring windows is served by the caches.  Each window
// value is loaded and converted once.  (The form before staged the window in
// LDS as fp32 and split the domain rows over the waves, every wave reading the
// whole window back: 47 us for 32x56x56x256 -> 157 MB of V in bf16, alpha' = 7,
// against 32 us now, 6.5 TB/s; 28 against 18 us for 32x28x28x512; 31 against 23
// us for the 3-channel 224x224 image; 14 against 7 us for 6x75x91x72 in fp16.)
#pragma once

#include <type_traits>
#include <utility>

#include "coefs.hpp"
#include "device_common.hpp"
#include "kernels.hpp"
#include "launch_split.hpp"

namespace wg {

// What a launch of the register form covers: whole images, or a band of tile
// rows of one image (launch_split.hpp).
// The geometry that it gets has the rows of pixels of an image or the band as H.
struct InputMap {
    FastDiv per_tile, tw, th;   // divisors: threads per tile, tiles per row, tile rows of an image or the band
    int64_t threads;            // (tile, run) pairs of this launch
    uint32_t xbytes;            // bytes of its pixels (at most kInMaxBytes)
    int64_t plane;              // bytes of a plane of V (all images)
};
// kInTop: whole images, or the band at the top of one; its first window row is the
// padding above it.  kInBelow: a band below, whose first window row is its first row
// of pixels (apart from kInTop because a run-time row was enough to make the code of
// 10x10 windows with alpha' = 10 in fp32 spill: 221 thousand threads 28 -> 39 us).
// kInFar: 64-bit addresses.
enum InputPart { kInTop, kInBelow, kInFar };

// VEC: channels per thread (2: 4-byte accesses of 16-bit pairs, C even; 1: one channel)
template <typename Elem, int VEC> struct InRun;
template <> struct InRun<float, 1> {
    using Bits = uint32_t;
    static __device__ __forceinline__ void unpack(Bits b, float* f) { f[0] = __uint_as_float(b); }
    static __device__ __forceinline__ Bits pack(const float* f) { return __float_as_uint(f[0]); }
    static __device__ __forceinline__ Bits load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
        return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
};
template <> struct InRun<bf16_t, 2> {
    using Bits = uint32_t;
    static __device__ __forceinline__ void unpack(Bits b, float* f) {
        f[0] = __uint_as_float(b << 16);
        f[1] = __uint_as_float(b & 0xffff0000u);
    }
    static __device__ __forceinline__ Bits pack(const float* f) {
        return static_cast<uint32_t>(Storage<bf16_t>::from_f32(f[0]).bits) |
               (static_cast<uint32_t>(Storage<bf16_t>::from_f32(f[1]).bits) << 16);
    }
    static __device__ __forceinline__ Bits load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
        return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
};
template <> struct InRun<_Float16, 2> {
    using Bits = uint32_t;
    static __device__ __forceinline__ void unpack(Bits b, float* f) {
        f[0] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(b)));
        f[1] = static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(b >> 16)));
    }
    static __device__ __forceinline__ Bits pack(const float* f) {
        return static_cast<uint32_t>(__builtin_bit_cast(uint16_t, Storage<_Float16>::from_f32(f[0]))) |
               (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, Storage<_Float16>::from_f32(f[1]))) << 16);
    }
    static __device__ __forceinline__ Bits load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
        return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
    }
};
template <typename Elem> struct InRun16 {
    using Bits = uint16_t;
    static __device__ __forceinline__ void unpack(Bits b, float* f) {
        f[0] = Storage<Elem>::to_f32(__builtin_bit_cast(Elem, b));
    }
    static __device__ __forceinline__ Bits pack(const float* f) {
        return __builtin_bit_cast(uint16_t, Storage<Elem>::from_f32(f[0]));
    }
    static __device__ __forceinline__ Bits load(__amdgpu_buffer_rsrc_t r, uint32_t off) {
        return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
    }
};
template <> struct InRun<bf16_t, 1> : InRun16<bf16_t> {};
template <> struct InRun<_Float16, 1> : InRun16<_Float16> {};

// Both passes for the domain rows A0 .. A1-1.  RELU: of ReLU(x), the elementwise
// step between two layers, applied as the window is read.
template <typename Elem, int TT, int ALPHA, class CO, int VEC, bool RELU, int A0, int A1>
__device__ __forceinline__ void input_regs_rows(const InputTable& tab, const typename InRun<Elem, VEC>::Bits (&d)[TT][TT],
                                                unsigned char* out, uint32_t lo, int64_t plane) {
    using R = InRun<Elem, VEC>;
    using Bits = typename R::Bits;
    constexpr int NR = A1 - A0;
    float W1[NR][TT][VEC];
#pragma unroll
    for (int v = 0; v < TT; ++v) {
        float col[TT][VEC];
#pragma unroll
        for (int u = 0; u < TT; ++u) {
            R::unpack(d[v][u], col[u]);
            if constexpr (RELU) {
#pragma unroll
                for (int q = 0; q < VEC; ++q) col[u][q] = col[u][q] > 0.0f ? col[u][q] : 0.0f;   // NaN and -0 give +0
            }
        }
#pragma unroll
        for (int a = 0; a < NR; ++a)
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                float acc = 0.0f;
#pragma unroll
                for (int u = 0; u < TT; ++u) acc = term<CO>(CO::bt(tab, (A0 + a) * TT + u), col[u][q], acc);
                W1[a][v][q] = acc;
            }
    }
#pragma unroll
    for (int a = 0; a < NR; ++a)
#pragma unroll
        for (int b = 0; b < ALPHA; ++b) {
            float f[VEC];
#pragma unroll
            for (int q = 0; q < VEC; ++q) {
                float acc = 0.0f;
#pragma unroll
                for (int v = 0; v < TT; ++v) acc = term<CO>(CO::bt(tab, b * TT + v), W1[a][v][q], acc);
                f[q] = acc;
            }
            *reinterpret_cast<Bits*>(out + ((A0 + a) * ALPHA + b) * plane + lo) = R::pack(f);
        }
}
template <typename Elem, int TT, int ALPHA, class CO, int VEC, bool RELU, int kR, int... Gs>
__device__ __forceinline__ void input_regs_groups(const InputTable& tab, const typename InRun<Elem, VEC>::Bits (&d)[TT][TT],
                                                  unsigned char* out, uint32_t lo, int64_t plane, int g,
                                                  std::integer_sequence<int, Gs...>) {
    auto one = [&](auto gc) __attribute__((always_inline)) {
        constexpr int a0 = decltype(gc)::value * kR, a1 = a0 + kR < ALPHA ? a0 + kR : ALPHA;
        if constexpr (a0 < a1)
            if (g == decltype(gc)::value) input_regs_rows<Elem, TT, ALPHA, CO, VEC, RELU, a0, a1>(tab, d, out, lo, plane);
    };
    (one(std::integral_constant<int, Gs>{}), ...);
}

// The window (columns first: a column's loads are issued together) and the
// thread's place in V.
//
// 32-bit offsets through a buffer descriptor (at most kInMaxBytes of pixels); a
// row or column outside the image gets an offset past every record, so its
// loads return zero without a branch (valid sums stay below 2^30).
template <typename Elem, int TT, int VEC, InputPart PART>
__device__ __forceinline__ void input_window(const Elem* __restrict__ x, const Geometry& geo, const InputMap& mp,
                                             uint32_t gid, typename InRun<Elem, VEC>::Bits (&d)[TT][TT]) {
    constexpr int ES = static_cast<int>(sizeof(Elem));
    constexpr int m = TT - 2;
    const uint32_t tile = fast_div(gid, mp.per_tile);
    const int c = static_cast<int>(gid - tile * mp.per_tile.d) * VEC;
    const uint32_t row = fast_div(tile, mp.tw);
    const int tx = static_cast<int>(tile - row * mp.tw.d);
    const uint32_t n = fast_div(row, mp.th);
    const int ty = static_cast<int>(row - n * mp.th.d);
    const int H = static_cast<int>(geo.H), W = static_cast<int>(geo.W), C = static_cast<int>(geo.C);
    const auto rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<Elem*>(x), static_cast<short>(0),
                                                      static_cast<int>(mp.xbytes), static_cast<int>(kRsrcWord3));
    uint32_t ro[TT], co[TT];
#pragma unroll
    for (int u = 0; u < TT; ++u) {
        const int hr = ty * m + u - (PART == kInTop ? 1 : 0);
        ro[u] = hr >= 0 && hr < H ? (n * static_cast<uint32_t>(H) + static_cast<uint32_t>(hr)) *
                                        static_cast<uint32_t>(W * C * ES)
                                  : 0x80000000u;
    }
#pragma unroll
    for (int v = 0; v < TT; ++v) {
        const int wc = tx * m - 1 + v;
        co[v] = wc >= 0 && wc < W && c < C ? static_cast<uint32_t>((wc * C + c) * ES) : 0x40000000u;
    }
#pragma unroll
    for (int v = 0; v < TT; ++v)
#pragma unroll
        for (int u = 0; u < TT; ++u) d[v][u] = InRun<Elem, VEC>::load(rx, ro[u] + co[v]);
}

// Images of which one tile row's pixels exceed kInMaxBytes: 64-bit addresses,
// loads behind their bounds.
template <typename Elem, int TT, int VEC>
__device__ __forceinline__ void input_window_big(const Elem* __restrict__ x, const Geometry& geo, int64_t gid,
                                                 typename InRun<Elem, VEC>::Bits (&d)[TT][TT]) {
    using Bits = typename InRun<Elem, VEC>::Bits;
    const int64_t runs = geo.Cp / VEC;
    const int64_t tile = gid / runs, c = (gid - tile * runs) * VEC;
    const int64_t tx = tile % geo.tw, ty = (tile / geo.tw) % geo.th, n = tile / (geo.tw * geo.th);
#pragma unroll
    for (int v = 0; v < TT; ++v)
#pragma unroll
        for (int u = 0; u < TT; ++u) {
            const int64_t hr = ty * (TT - 2) - 1 + u, wc = tx * (TT - 2) - 1 + v;
            const bool in = hr >= 0 && hr < geo.H && wc >= 0 && wc < geo.W && c < geo.C;
            const Elem* src = x + ((n * geo.H + hr) * geo.W + wc) * geo.C + c;
            d[v][u] = in ? *reinterpret_cast<const Bits*>(src) : Bits(0);
        }
}

template <typename Elem, int TT, int ALPHA, class CO, int VEC, int RG, InputPart PART, bool RELU>
__device__ __forceinline__ void input_regs_unit(const InputTable& tab, const Elem* __restrict__ x,
                                                unsigned char* __restrict__ V, const Geometry& geo,
                                                const InputMap& mp, int64_t bid, int64_t G) {
    using R = InRun<Elem, VEC>;
    using Bits = typename R::Bits;
    constexpr int ES = static_cast<int>(sizeof(Elem));
    // XCD-aware numbering: the hardware deals workgroup ids round-robin to the
    // 8 XCDs; giving each XCD a contiguous run keeps neighbouring tiles, whose
    // windows overlap, in the same L2
    const int64_t xcd = bid % 8;
    const int64_t unit = xcd * (G / 8) + (xcd < G % 8 ? xcd : G % 8) + bid / 8;
    const int group = RG == 1 ? 0 : static_cast<int>(unit % RG);   // row group of this workgroup
    const int64_t base = unit / RG * kInBlock;
    const int64_t gid = base + threadIdx.x;
    if (gid >= mp.threads) return;
    Bits d[TT][TT];
    if constexpr (PART == kInFar) input_window_big<Elem, TT, VEC>(x, geo, gid, d);
    else input_window<Elem, TT, VEC, PART>(x, geo, mp, static_cast<uint32_t>(gid), d);
    unsigned char* out = V + base * (VEC * ES);
    const uint32_t lo = threadIdx.x * (VEC * ES);
    if constexpr (RG == 1) {
        input_regs_rows<Elem, TT, ALPHA, CO, VEC, RELU, 0, ALPHA>(tab, d, out, lo, mp.plane);
    } else {
        constexpr int kR = (ALPHA + RG - 1) / RG;
        input_regs_groups<Elem, TT, ALPHA, CO, VEC, RELU, kR>(tab, d, out, lo, mp.plane, group,
                                                        std::make_integer_sequence<int, RG>{});
    }
}

}  // namespace wg
