// Operations around the Winograd layer on gfx950:
//   * ReLU and 2x2 stride-2 max-pooling between the convolutions of a CNN
//     (the VGG-16 stack of the experiments of Section 3.2 of Barabasz &
//     Gregg, arXiv 1905.05233);
//   * a float64 direct convolution, the reference against which Section 3.1
//     measures the error of a Winograd convolution computed in lower
//     precision;
//   * the two sums of squares that the relative L2 error of a result against
//     such a reference needs, reduced in float64 in a fixed order.
// None of these is on the Winograd path itself; they keep the stack and the
// error studies on the device.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "device_common.hpp"
#include "kernels.hpp"
#include "launch_split.hpp"

namespace wg {

namespace {

constexpr int kOpBlock = 256;

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// 16 bytes as non-temporal (streaming) accesses: the input is read once and
// the output is read once, by the next layer's transforms; kept out of the
// caches, they leave the last-level cache to the next layer's V and U (a
// VGG-16 pass at N = 32: 1.78 against 1.82 ms of convolution time for the
// stores, 1.73 against 1.74 ms for the loads)
__device__ __forceinline__ void store16_nt(void* dst, const void* src) {
    __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(src), reinterpret_cast<u32x4*>(dst));
}
__device__ __forceinline__ u32x4 load16_nt(const void* src) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
}

template <typename Elem>
__device__ __forceinline__ float relu(Elem v) {
    const float f = Storage<Elem>::to_f32(v);
    return f > 0.0f ? f : 0.0f;   // NaN and -0 give +0
}

// y = ReLU(x), elementwise over n values; vec values per thread (a 16-byte
// run when the whole tensor is made of such runs, else one value).
template <typename Elem, int VEC>
__global__ __launch_bounds__(kOpBlock) void relu_kernel(const Elem* __restrict__ x, Elem* __restrict__ y,
                                                        int64_t n) {
    using S = Storage<Elem>;
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * kOpBlock + threadIdx.x) * VEC;
    if (i >= n) return;
    Elem e[VEC];
    if constexpr (VEC * sizeof(Elem) == 16) {
        *reinterpret_cast<u32x4*>(e) = load16_nt(x + i);
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) e[q] = x[i + q];
    }
#pragma unroll
    for (int q = 0; q < VEC; ++q) e[q] = S::from_f32(relu(e[q]));
    if constexpr (VEC * sizeof(Elem) == 16) {
        store16_nt(y + i, e);
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) y[i + q] = e[q];
    }
}

// y[n][i][j][c] = max over the 2x2 window at (2i, 2j) of ReLU(x); one thread
// per (output pixel, run of VEC channels), channels fastest (coalesced).
template <typename Elem, int VEC>
__global__ __launch_bounds__(kOpBlock) void relu_pool_kernel(const Elem* __restrict__ x, Elem* __restrict__ y,
                                                             int64_t N, int64_t H, int64_t W, int64_t C) {
    using S = Storage<Elem>;
    const int64_t Ho = H / 2, Wo = W / 2, runs = C / VEC;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kOpBlock + threadIdx.x;
    if (gid >= N * Ho * Wo * runs) return;
    const int64_t c = (gid % runs) * VEC;
    const int64_t pix = gid / runs;
    const int64_t j = pix % Wo, i = (pix / Wo) % Ho, n = pix / (Wo * Ho);
    float best[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) best[q] = 0.0f;
#pragma unroll
    for (int di = 0; di < 2; ++di)
#pragma unroll
        for (int dj = 0; dj < 2; ++dj) {
            const Elem* src = x + ((n * H + 2 * i + di) * W + 2 * j + dj) * C + c;
            Elem e[VEC];
            if constexpr (VEC * sizeof(Elem) == 16) {
                *reinterpret_cast<u32x4*>(e) = load16_nt(src);
            } else {
#pragma unroll
                for (int q = 0; q < VEC; ++q) e[q] = src[q];
            }
#pragma unroll
            for (int q = 0; q < VEC; ++q) best[q] = fmaxf(best[q], relu(e[q]));
        }
    Elem o[VEC];
#pragma unroll
    for (int q = 0; q < VEC; ++q) o[q] = S::from_f32(best[q]);
    Elem* dst = y + pix * C + c;
    if constexpr (VEC * sizeof(Elem) == 16) {
        store16_nt(dst, o);
    } else {
#pragma unroll
        for (int q = 0; q < VEC; ++q) dst[q] = o[q];
    }
}

// yd[n][h][v][k] = sum_{i<KH, j<3, c} w[k][i][j][c] x[n][h + i - KH/2][v + j - 1][c]
// in float64 (zero outside the image).  One thread per output, output
// channels fastest: the 64 lanes of a wave share their input pixel.
template <typename Elem, int KH>
__device__ __forceinline__ double direct_f64_one(const Elem* __restrict__ x, const Elem* __restrict__ w, int64_t pix,
                                                 int64_t k, int64_t H, int64_t W, int64_t C) {
    using S = Storage<Elem>;
    const int64_t v = pix % W, h = (pix / W) % H, n = pix / (W * H);
    double acc = 0.0;
    for (int i = 0; i < KH; ++i) {
        const int64_t hh = h + i - KH / 2;
        if (hh < 0 || hh >= H) continue;
        for (int j = 0; j < 3; ++j) {
            const int64_t vv = v + j - 1;
            if (vv < 0 || vv >= W) continue;
            const Elem* xs = x + ((n * H + hh) * W + vv) * C;
            const Elem* ws = w + ((k * KH + i) * 3 + j) * C;
            for (int64_t c = 0; c < C; ++c)
                acc = fma(static_cast<double>(S::to_f32(ws[c])), static_cast<double>(S::to_f32(xs[c])), acc);
        }
    }
    return acc;
}

template <typename Elem, int KH>
__global__ __launch_bounds__(kOpBlock) void direct_f64_kernel(const Elem* __restrict__ x, const Elem* __restrict__ w,
                                                              double* __restrict__ yd, int64_t N, int64_t H, int64_t W,
                                                              int64_t C, int64_t K) {
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kOpBlock + threadIdx.x;
    if (gid >= N * H * W * K) return;
    yd[gid] = direct_f64_one<Elem, KH>(x, w, gid / K, gid % K, H, W, C);
}

// The same as a matrix product on the float64 matrix cores, for layers with
// enough output channels and taps: y [pixels][K] = X [pixels][R] W^T [R][K] with
// R = KH 3 C, X's row the pixel's window (W is contiguous in R).  A workgroup of
// four waves computes BM x BN outputs, each wave 16 WT x 16 WT of them in tiles
// of v_mfma_f64_16x16x4_f64.  Chunks of 32 values of R are widened to fp32
// (exact), staged in double-buffered LDS and widened to float64 as fragments;
// the next chunk's loads, branch-free through buffer descriptors, are in flight
// during the current one's products.  Within 16 values lane group g of a wave
// takes the values 4 g .. 4 g + 3, one per instruction, the same on both
// operands.  Taps outside the image enter as x = 0, which a finite weight turns
// into nothing; a block that meets an infinite or NaN weight recomputes its
// outputs with those taps left out.
//
// What bounds it: the matrix cores (64 clocks per instruction), and for layers of
// few blocks the latency of a chunk.  2x56x56, 128 -> 128 (1.85 GFLOP): 2650 us
// with one thread per output, 64 us here (29 TFLOP/s; 196 blocks of four waves
// leave 60 of the 256 CUs idle); 2x28x28, 512 -> 512: 13900 and 242 us.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr int kF64Chunk = 32;
constexpr int kF64Row = kF64Chunk + 4;   // floats per LDS row: 16-byte aligned, off the bank period

struct F64Geometry {
    int64_t H, W, C, K, pixels;
    int R;
    FastDiv c;                  // by C
    uint32_t xbytes, wbytes;    // both below kOob
};

// Four consecutive values of R as loaded (V4: one aligned load), and widened to
// fp32.  The two are apart so that the wait for a load comes where the values
// are parked, behind the products: widened at the load, 16-bit layers waited
// ahead of every chunk's products (2x56x56, 128 -> 128 in bf16 72.7 us, now 63.8).
template <typename Elem, bool V4> struct Run4 {
    using Bits = std::conditional_t<V4 && sizeof(Elem) == 2, u32x2, u32x4>;
    static __device__ __forceinline__ Bits load(__amdgpu_buffer_rsrc_t r, const uint32_t (&off)[4]) {
        if constexpr (V4 && sizeof(Elem) == 4) {
            return __builtin_amdgcn_raw_buffer_load_b128(r, off[0], 0, 0);
        } else if constexpr (V4) {
            return __builtin_amdgcn_raw_buffer_load_b64(r, off[0], 0, 0);
        } else {
            Bits b;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if constexpr (sizeof(Elem) == 4) b[e] = __builtin_amdgcn_raw_buffer_load_b32(r, off[e], 0, 0);
                else b[e] = static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(r, off[e], 0, 0));
            }
            return b;
        }
    }
    static __device__ __forceinline__ f32x4 widen(const Bits& b) {
        using S = Storage<Elem>;
        f32x4 f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (sizeof(Elem) == 4) f[e] = __uint_as_float(b[e]);
            else if constexpr (V4) f[e] = S::to_f32(__builtin_bit_cast(Elem, static_cast<uint16_t>(b[e >> 1] >> (16 * (e & 1)))));
            else f[e] = S::to_f32(__builtin_bit_cast(Elem, static_cast<uint16_t>(b[e])));
        }
        return f;
    }
};

template <typename Elem, int KH, int BM, int BN, int WT, bool V4>
__global__ __launch_bounds__(256) void direct_f64_mfma_kernel(const Elem* __restrict__ x, const Elem* __restrict__ w,
                                                              double* __restrict__ yd, F64Geometry g) {
    constexpr int ES = static_cast<int>(sizeof(Elem));
    constexpr int kWN = BN / (16 * WT);        // waves along the output channels
    static_assert((BM / (16 * WT)) * kWN == 4, "four waves");
    static_assert(WT == 1 || WT == 2, "the wait behind the products names its sums");
    constexpr int kXI = BM / 32, kWI = BN / 32;   // row groups of 32 that a thread loads for
    __shared__ __attribute__((aligned(16))) float st[2][(BM + BN) * kF64Row];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / kWN, wn = wave % kWN;
    const int64_t m0 = static_cast<int64_t>(blockIdx.x) * BM;
    const int64_t n0 = static_cast<int64_t>(blockIdx.y) * BN;
    const auto rx = make_rsrc(x, g.xbytes);
    const auto rw = make_rsrc(w, g.wbytes);
    // staging: thread t loads values 4 (t % 8) .. + 3 of the chunk for rows t / 8 + 32 i
    const int q4 = (tid & 7) * 4;
    const int row0 = tid >> 3;
    uint32_t xoff[kXI], woff[kWI];
    int xh[kXI], xw[kXI];
#pragma unroll
    for (int i = 0; i < kXI; ++i) {
        const int64_t pix = m0 + row0 + 32 * i;
        const int64_t pp = pix < g.pixels ? pix : 0;
        xw[i] = static_cast<int>(pp % g.W);
        // rows past the last pixel: a height no tap reaches from inside the image
        xh[i] = pix < g.pixels ? static_cast<int>((pp / g.W) % g.H) : -4;
        xoff[i] = static_cast<uint32_t>(pp * g.C * ES);
    }
#pragma unroll
    for (int i = 0; i < kWI; ++i) {
        const int64_t k = n0 + row0 + 32 * i;
        woff[i] = k < g.K ? static_cast<uint32_t>(k * g.R * ES) : kOob;
    }
    using Run = Run4<Elem, V4>;
    typename Run::Bits xr[kXI], wr[kWI];
    bool odd = false;   // an infinite or NaN weight
    auto load = [&](int r0) __attribute__((always_inline)) {
        int di[4], dj[4];
        uint32_t dx[4];   // byte offset of the tap and channel from the row's pixel (modulo 2^32)
        bool in[4];
#pragma unroll
        for (int e = 0; e < (V4 ? 1 : 4); ++e) {
            const int r = r0 + q4 + e;
            in[e] = r < g.R;
            const int tap = static_cast<int>(fast_div(static_cast<uint32_t>(r), g.c));
            di[e] = KH == 3 ? tap / 3 - 1 : 0;
            dj[e] = (KH == 3 ? tap % 3 : tap) - 1;
            dx[e] = static_cast<uint32_t>(((static_cast<int64_t>(di[e]) * g.W + dj[e]) * g.C + (r - tap * static_cast<int>(g.C))) * ES);
        }
#pragma unroll
        for (int i = 0; i < kXI; ++i) {
            uint32_t off[4];
#pragma unroll
            for (int e = 0; e < (V4 ? 1 : 4); ++e) {
                const uint32_t h = static_cast<uint32_t>(xh[i] + di[e]), v = static_cast<uint32_t>(xw[i] + dj[e]);
                // & and not &&: a select, no branch between the loads
                const bool ok = in[e] & (h < static_cast<uint32_t>(g.H)) & (v < static_cast<uint32_t>(g.W));
                off[e] = ok ? xoff[i] + dx[e] : kOob;
            }
            xr[i] = Run::load(rx, off);
        }
#pragma unroll
        for (int i = 0; i < kWI; ++i) {
            uint32_t off[4];
#pragma unroll
            for (int e = 0; e < (V4 ? 1 : 4); ++e)
                off[e] = in[e] & (woff[i] != kOob) ? woff[i] + static_cast<uint32_t>((r0 + q4 + e) * ES) : kOob;
            wr[i] = Run::load(rw, off);
        }
    };
    auto park = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kXI; ++i) *reinterpret_cast<f32x4*>(&st[buf][(row0 + 32 * i) * kF64Row + q4]) = Run::widen(xr[i]);
#pragma unroll
        for (int i = 0; i < kWI; ++i) {
            const f32x4 f = Run::widen(wr[i]);
            *reinterpret_cast<f32x4*>(&st[buf][(BM + row0 + 32 * i) * kF64Row + q4]) = f;
#pragma unroll
            for (int e = 0; e < 4; ++e) odd |= !(__builtin_fabsf(f[e]) < __builtin_inff());
        }
    };
    f64x4 acc[WT][WT];
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int l16 = lane & 15, grp = lane >> 4;
    load(0);
    park(0);
    __syncthreads();
    int buf = 0;
    for (int r0 = 0; r0 < g.R; r0 += kF64Chunk) {
        const bool more = r0 + kF64Chunk < g.R;
        if (more) load(r0 + kF64Chunk);
        f64x4 part[WT][WT];
#pragma unroll
        for (int s = 0; s < kF64Chunk / 16; ++s) {
            f32x4 a[WT], b[WT];
#pragma unroll
            for (int i = 0; i < WT; ++i) {
                a[i] = *reinterpret_cast<const f32x4*>(&st[buf][(wm * 16 * WT + i * 16 + l16) * kF64Row + s * 16 + grp * 4]);
                b[i] = *reinterpret_cast<const f32x4*>(&st[buf][(BM + wn * 16 * WT + i * 16 + l16) * kF64Row + s * 16 + grp * 4]);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < WT; ++i)
#pragma unroll
                    for (int j = 0; j < WT; ++j)
                        part[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                            static_cast<double>(a[i][e]), static_cast<double>(b[j][e]),
                            s == 0 && e == 0 ? f64x4{0.0, 0.0, 0.0, 0.0} : part[i][j], 0, 0, 0);
        }
        // Wait out the last product before its result is read (the compiler
        // keeps 19 wait states between the two on gfx950).  Without this wait
        // it was seen to place a copy of a result's last register ahead of its
        // own wait states, where the block ends in a branch (an accvgpr_read two
        // states behind the product; rows 12 .. 15 of a tile came out wrong).
        // The sums are operands of the wait, in the registers that the products
        // write, so what reads them comes behind it;
        // tests/test_f64_waits.py checks the code of every instance.
        if constexpr (WT == 1)
            asm volatile("s_nop 15\n\ts_nop 2" : "+a"(part[0][0]));
        else
            asm volatile("s_nop 15\n\ts_nop 2" : "+a"(part[0][0]), "+a"(part[0][1]), "+a"(part[1][0]), "+a"(part[1][1]));
        // a chunk's sum, then the chunks': fewer roundings than one chain over R
#pragma unroll
        for (int i = 0; i < WT; ++i)
#pragma unroll
            for (int j = 0; j < WT; ++j) acc[i][j] += part[i][j];
        if (more) {
            park(buf ^ 1);
            __syncthreads();
            buf ^= 1;
        }
    }
    const bool recompute = __syncthreads_or(odd ? 1 : 0) != 0;
    // lane l, value r of a tile: row 4 r + l / 16, column l % 16
#pragma unroll
    for (int i = 0; i < WT; ++i)
#pragma unroll
        for (int j = 0; j < WT; ++j) {
            const int64_t k = n0 + wn * 16 * WT + j * 16 + l16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t pix = m0 + wm * 16 * WT + i * 16 + 4 * r + grp;
                if (pix >= g.pixels || k >= g.K) continue;
                yd[pix * g.K + k] = recompute ? direct_f64_one<Elem, KH>(x, w, pix, k, g.H, g.W, g.C) : acc[i][j][r];
            }
        }
}

template <typename Elem, int BM, int BN, int WT>
hipError_t launch_f64_mfma(const F64Geometry& g, const Elem* x, const Elem* w, double* y, int kh, hipStream_t stream) {
    const dim3 grid(static_cast<unsigned>((g.pixels + BM - 1) / BM), static_cast<unsigned>((g.K + BN - 1) / BN));
#define WG_F64(KH, V4) \
    hipLaunchKernelGGL((direct_f64_mfma_kernel<Elem, KH, BM, BN, WT, V4>), grid, dim3(256), 0, stream, x, w, y, g)
    const bool v4 = g.C % 4 == 0;
    if (kh == 3 && v4) WG_F64(3, true);
    else if (kh == 3) WG_F64(3, false);
    else if (v4) WG_F64(1, true);
    else WG_F64(1, false);
#undef WG_F64
    return hipGetLastError();
}

// Sums of (y - ref)^2 and ref^2 over n values in float64: each of the
// kSumBlocks blocks strides over the values and reduces its part in LDS in a
// fixed order into sums[2 + 2 b], sums[3 + 2 b]; one block then adds the
// partials in block order into sums[0], sums[1].  Deterministic.
constexpr int kSumBlocks = 256;

template <typename Elem>
__global__ __launch_bounds__(kOpBlock) void sq_sums_partial(const Elem* __restrict__ y, const double* __restrict__ ref,
                                                            int64_t n, double* __restrict__ sums) {
    using S = Storage<Elem>;
    __shared__ double se[kOpBlock], sr[kOpBlock];
    double e2 = 0.0, r2 = 0.0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kOpBlock + threadIdx.x; i < n;
         i += static_cast<int64_t>(kSumBlocks) * kOpBlock) {
        const double r = ref[i];
        const double d = static_cast<double>(S::to_f32(y[i])) - r;
        e2 = fma(d, d, e2);
        r2 = fma(r, r, r2);
    }
    se[threadIdx.x] = e2;
    sr[threadIdx.x] = r2;
    __syncthreads();
    for (int s = kOpBlock / 2; s > 0; s >>= 1) {
        if (static_cast<int>(threadIdx.x) < s) {
            se[threadIdx.x] += se[threadIdx.x + s];
            sr[threadIdx.x] += sr[threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        sums[2 + 2 * blockIdx.x] = se[0];
        sums[3 + 2 * blockIdx.x] = sr[0];
    }
}

__global__ __launch_bounds__(64) void sq_sums_final(double* __restrict__ sums) {
    if (threadIdx.x != 0) return;
    double e2 = 0.0, r2 = 0.0;
    for (int b = 0; b < kSumBlocks; ++b) {
        e2 += sums[2 + 2 * b];
        r2 += sums[3 + 2 * b];
    }
    sums[0] = e2;
    sums[1] = r2;
}

inline unsigned op_blocks(int64_t n) { return static_cast<unsigned>((n + kOpBlock - 1) / kOpBlock); }

}  // namespace

template <int D>
hipError_t launch_relu_pool_t(const void* x, void* y, int64_t N, int64_t H, int64_t W, int64_t C, bool pool,
                              hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    constexpr int kVec = 16 / static_cast<int>(sizeof(Elem));
    const auto* xp = static_cast<const Elem*>(x);
    auto* yp = static_cast<Elem*>(y);
    const bool vec = C % kVec == 0;
    if (!pool) {
        const int64_t n = N * H * W * C;
        const int64_t threads = vec ? n / kVec : n;
        if ((threads + kOpBlock - 1) / kOpBlock > 0x7fffffff) return hipErrorInvalidValue;
        if (vec)
            hipLaunchKernelGGL((relu_kernel<Elem, kVec>), dim3(op_blocks(threads)), dim3(kOpBlock), 0, stream, xp, yp, n);
        else
            hipLaunchKernelGGL((relu_kernel<Elem, 1>), dim3(op_blocks(threads)), dim3(kOpBlock), 0, stream, xp, yp, n);
        return hipGetLastError();
    }
    const int64_t threads = N * (H / 2) * (W / 2) * (vec ? C / kVec : C);
    if (threads == 0) return hipSuccess;
    if ((threads + kOpBlock - 1) / kOpBlock > 0x7fffffff) return hipErrorInvalidValue;
    if (vec)
        hipLaunchKernelGGL((relu_pool_kernel<Elem, kVec>), dim3(op_blocks(threads)), dim3(kOpBlock), 0, stream, xp, yp,
                           N, H, W, C);
    else
        hipLaunchKernelGGL((relu_pool_kernel<Elem, 1>), dim3(op_blocks(threads)), dim3(kOpBlock), 0, stream, xp, yp, N,
                           H, W, C);
    return hipGetLastError();
}

template <int D>
hipError_t launch_direct_f64_t(const void* x, const void* w, double* y, int64_t N, int64_t H, int64_t W, int64_t C,
                               int64_t K, int kh, hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    const int64_t n = N * H * W * K;
    if ((n + kOpBlock - 1) / kOpBlock > 0x7fffffff) return hipErrorInvalidValue;
    const auto* xp = static_cast<const Elem*>(x);
    const auto* wp = static_cast<const Elem*>(w);
    const int64_t R = static_cast<int64_t>(kh) * 3 * C, pixels = N * H * W, es = sizeof(Elem);
    const F64Form form = f64_form(pixels, C, K, kh * 3, es, device_cu_count());
    if (form != kF64PerOutput) {
        const F64Geometry g{H, W, C, K, pixels, static_cast<int>(R), make_fastdiv(C),
                            static_cast<uint32_t>(pixels * C * es), static_cast<uint32_t>(K * R * es)};
        if (form == kF64Block32) return launch_f64_mfma<Elem, 32, 32, 1>(g, xp, wp, y, kh, stream);
        if (form == kF64Block64) return launch_f64_mfma<Elem, 64, 64, 2>(g, xp, wp, y, kh, stream);
        return launch_f64_mfma<Elem, 128, 32, 2>(g, xp, wp, y, kh, stream);
    }
    if (kh == 3)
        hipLaunchKernelGGL((direct_f64_kernel<Elem, 3>), dim3(op_blocks(n)), dim3(kOpBlock), 0, stream, xp, wp, y, N, H,
                           W, C, K);
    else
        hipLaunchKernelGGL((direct_f64_kernel<Elem, 1>), dim3(op_blocks(n)), dim3(kOpBlock), 0, stream, xp, wp, y, N, H,
                           W, C, K);
    return hipGetLastError();
}

template <int D>
hipError_t launch_sq_sums_t(const void* y, const double* ref, int64_t n, double* sums, hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    hipLaunchKernelGGL((sq_sums_partial<Elem>), dim3(kSumBlocks), dim3(kOpBlock), 0, stream,
                       static_cast<const Elem*>(y), ref, n, sums);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sq_sums_final, dim3(1), dim3(64), 0, stream, sums);
    return hipGetLastError();
}

template hipError_t launch_relu_pool_t<0>(const void*, void*, int64_t, int64_t, int64_t, int64_t, bool, hipStream_t);
template hipError_t launch_relu_pool_t<1>(const void*, void*, int64_t, int64_t, int64_t, int64_t, bool, hipStream_t);
template hipError_t launch_relu_pool_t<2>(const void*, void*, int64_t, int64_t, int64_t, int64_t, bool, hipStream_t);
template hipError_t launch_direct_f64_t<0>(const void*, const void*, double*, int64_t, int64_t, int64_t, int64_t,
                                           int64_t, int, hipStream_t);
template hipError_t launch_direct_f64_t<1>(const void*, const void*, double*, int64_t, int64_t, int64_t, int64_t,
                                           int64_t, int, hipStream_t);
template hipError_t launch_direct_f64_t<2>(const void*, const void*, double*, int64_t, int64_t, int64_t, int64_t,
                                           int64_t, int, hipStream_t);
template hipError_t launch_sq_sums_t<0>(const void*, const double*, int64_t, double*, hipStream_t);
template hipError_t launch_sq_sums_t<1>(const void*, const double*, int64_t, double*, hipStream_t);
template hipError_t launch_sq_sums_t<2>(const void*, const double*, int64_t, double*, hipStream_t);

}  // namespace wg
