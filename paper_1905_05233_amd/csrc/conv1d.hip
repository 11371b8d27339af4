// 1D Winograd convolution F(m, 3) on gfx950: the one-dimensional form of the
// algorithm of Section 2 of Barabasz & Gregg (arXiv 1905.05233),
//     y = A^T [ (G g) (.) (B^T d) ],
// on input tiles d of m + 2 values overlapping by two, summed over input
// channels; Section 3.1 studies its error next to the 2D form.
//
// Layouts (channels last): x [N][1][L][C], w [K][1][3][C], y [N][1][L][K];
// U [alpha'][K][Cp], V [alpha'][T][Cp] (T = N * ceil(L / m), tile index
// t = n * ceil(L / m) + tx), M [alpha'][T][Kp] fp32.  The contraction is the
// 2D library's (alpha' planes instead of alpha'^2).
//
// Each transform is one 1D pass with the operation order of the 2D kernels:
// from zero, ascending index, one fused multiply-add per term in fp32, one
// rounding to the storage dtype at the store.  One thread per (tile or
// kernel, channel), channels fastest, so a wave's loads and stores sweep 64
// consecutive channels.  Loops run to the largest tile (16) and stop at the
// layer's t and alpha' by uniform conditions, so the register arrays keep
// compile-time indices and one instance serves every plan.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "device_common.hpp"
#include "kernels.hpp"
#include "launch_split.hpp"

namespace wg {

namespace {

constexpr int kBlock1d = 256;

// U[a][k][c] = sum_i G[a][i] g[k][i][c]
template <typename Elem>
__global__ __launch_bounds__(kBlock1d) void kernel_transform_1d(KernelTable tab, const Elem* __restrict__ w,
                                                                Elem* __restrict__ U, int64_t K, int64_t C,
                                                                int64_t Cp, int alpha) {
    using S = Storage<Elem>;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kBlock1d + threadIdx.x;
    if (gid >= K * Cp) return;
    const int64_t c = gid % Cp, k = gid / Cp;
    float g[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) g[i] = c < C ? S::to_f32(w[(k * 3 + i) * C + c]) : 0.0f;
#pragma unroll
    for (int a = 0; a < kMaxAlpha; ++a) {
        if (a >= alpha) break;
        float acc = 0.0f;
#pragma unroll
        for (int i = 0; i < 3; ++i) acc = __builtin_fmaf(tab.g[a * 3 + i], g[i], acc);
        U[(a * K + k) * Cp + c] = S::from_f32(acc);
    }
}

// V[a][t][c] = sum_u B^T[a][u] d[u], d the window of t values at tx*m - 1
template <typename Elem>
__global__ __launch_bounds__(kBlock1d) void input_transform_1d(InputTable tab, const Elem* __restrict__ x,
                                                               Elem* __restrict__ V, int64_t L, int64_t C, int64_t Cp,
                                                               int64_t tl, int64_t T, int m, int tt, int alpha) {
    using S = Storage<Elem>;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kBlock1d + threadIdx.x;
    if (gid >= T * Cp) return;
    const int64_t c = gid % Cp, t = gid / Cp;
    const int64_t tx = t % tl, n = t / tl;
    const int64_t l0 = tx * m - 1;
    float d[kMaxTile];
#pragma unroll
    for (int u = 0; u < kMaxTile; ++u) {
        const int64_t l = l0 + u;
        d[u] = (u < tt && c < C && l >= 0 && l < L) ? S::to_f32(x[(n * L + l) * C + c]) : 0.0f;
    }
#pragma unroll
    for (int a = 0; a < kMaxAlpha; ++a) {
        if (a >= alpha) break;
        float acc = 0.0f;
#pragma unroll
        for (int u = 0; u < kMaxTile; ++u) {
            if (u >= tt) break;
            acc = __builtin_fmaf(tab.bt[a * tt + u], d[u], acc);
        }
        V[(a * T + t) * Cp + c] = S::from_f32(acc);
    }
}

// y[n][tx*m + o][k] = sum_a A^T[o][a] M[a][t][k], stored inside L only
template <typename Elem>
__global__ __launch_bounds__(kBlock1d) void output_transform_1d(OutputTable tab, const float* __restrict__ M,
                                                                Elem* __restrict__ y, int64_t L, int64_t K, int64_t Kp,
                                                                int64_t tl, int64_t T, int m, int alpha) {
    using S = Storage<Elem>;
    const int64_t gid = static_cast<int64_t>(blockIdx.x) * kBlock1d + threadIdx.x;
    if (gid >= T * K) return;
    const int64_t k = gid % K, t = gid / K;
    const int64_t tx = t % tl, n = t / tl;
    float mv[kMaxAlpha];
#pragma unroll
    for (int a = 0; a < kMaxAlpha; ++a) mv[a] = a < alpha ? M[(a * T + t) * Kp + k] : 0.0f;
#pragma unroll
    for (int o = 0; o < kMaxTile; ++o) {
        const int64_t l = tx * m + o;
        if (o >= m || l >= L) break;
        float acc = 0.0f;
#pragma unroll
        for (int a = 0; a < kMaxAlpha; ++a) {
            if (a >= alpha) break;
            acc = __builtin_fmaf(tab.at[o * alpha + a], mv[a], acc);
        }
        y[(n * L + l) * K + k] = S::from_f32(acc);
    }
}

// ---------------------------------------------------------------------------
// Input transform, contraction and output transform in one kernel.
//
// The alpha' points of the 1D form leave room for all their sums in a wave's
// accumulators, so neither V nor M reaches memory: a workgroup of eight waves
// owns 16 kw output channels x 32 (8 / kw) tiles (kw = 8 waves side by side
// along the channels, or 4 where K <= 64) and walks the channels in chunks of 64
// bytes.  Per chunk each thread computes the alpha' V values of one (tile, 4
// bytes of channels) window, in the order of the stand-alone transform, into
// double-buffered LDS, while the last chunk's V goes through the matrix cores
// against U, whose fragments come straight from memory (U is small and stays in
// L2).  At the end a lane holds M of four consecutive channels of a tile for
// every point and applies A^T.
//
// What bounds it: the stores of y and the loads of U and of the windows, all
// cached.  16x4096, 128 -> 128 in fp16, alpha' = 7 (V 29 MB and M 59 MB crossed
// memory before): 86 us in four launches, 26 us in two now; in fp32 100 and 67 us.
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int k1dTiles = 64;             // most tiles of a block
constexpr int k1dMaxAlpha = 10;

template <int D>
__device__ __forceinline__ void mma_1d(const u32x4& a, const u32x4& b, f32x4& c) {
    static_assert(D != 0, "16-bit fragments");
    if constexpr (D == 1) {
        c = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    } else {
        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
}

struct Map1d {
    FastDiv tl;                  // tiles per row
    uint32_t xbytes;
    int kw, n_kb, rb, n_chunks, plane_u;   // plane_u: bytes of one point of U
};

template <int D, int TT, int ALPHA>
__global__ __launch_bounds__(64 * k1dWaves, (D != 0 && ALPHA <= 7 ? 4 : 2)) void conv1d_fused_kernel(
    const typename DTypeOf<D>::type* __restrict__ x, const unsigned char* __restrict__ U,
    typename DTypeOf<D>::type* __restrict__ y, InputTable itab, OutputTable otab, Geometry geo, Map1d mp) {
    using Elem = typename DTypeOf<D>::type;
    using S = Storage<Elem>;
    constexpr int ES = static_cast<int>(sizeof(Elem));
    constexpr int VEC = 4 / ES;                       // channels of a 4-byte run
    constexpr int MM = TT - 2;
    constexpr int kPoint = k1dTiles * k1dChunk;       // LDS bytes of one point's V
    __shared__ __attribute__((aligned(16))) unsigned char vb[2][ALPHA * kPoint];

    const int64_t G = gridDim.x, bid = blockIdx.x, xcd = bid % 8;
    const int64_t unit = xcd * (G / 8) + (xcd < G % 8 ? xcd : G % 8) + bid / 8;   // XCD-aware
    const int kb = static_cast<int>(unit % mp.n_kb);
    const int n_tiles = 32 * (k1dWaves / mp.kw);      // tiles of the block
    const int64_t t0 = unit / mp.n_kb * n_tiles;
    const int k0 = kb * 16 * mp.kw;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % mp.kw, wt = wave / mp.kw;
    const int grp = lane >> 4, l16 = lane & 15;
    const int C = static_cast<int>(geo.C), L = static_cast<int>(geo.W);
    const int T = static_cast<int>(geo.T), K = static_cast<int>(geo.K);

    // this thread's windows: 4-byte run tid % 16 of tiles tid / 16 and + 32
    const int run = tid & 15;
    const auto rx = make_rsrc(x, mp.xbytes);
    uint32_t xo[2];              // byte offset of the window's first position (modulo 2^32)
    int l0[2];                   // that position in the row; past every row for absent tiles
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t t = t0 + (tid >> 4) + 32 * i;
        const uint32_t tt = static_cast<uint32_t>(t < T ? t : 0);
        const uint32_t n = fast_div(tt, mp.tl);
        const int tx = static_cast<int>(tt - n * mp.tl.d);
        l0[i] = t < T ? tx * MM - 1 : 0x40000000;
        xo[i] = (n * static_cast<uint32_t>(L) + static_cast<uint32_t>(tx * MM - 1)) * static_cast<uint32_t>(C * ES);
    }
    const bool two = n_tiles == 64;
    // runs that straddle two positions (odd C in 16 bits) go element by element
    const bool pairs = (C * ES) % 4 == 0;
    uint32_t d[2][TT];
    auto load = [&](int ck) __attribute__((always_inline)) {
        const int c = ck * (k1dChunk / ES) + run * VEC;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (i == 0 || two)
#pragma unroll
            for (int u = 0; u < TT; ++u) {
                const int l = l0[i] + u;
                const bool in = l >= 0 && l < L && c < C;
                const uint32_t off = xo[i] + static_cast<uint32_t>((u * C + c) * ES);
                if (ES == 4 || pairs) {
                    d[i][u] = __builtin_amdgcn_raw_buffer_load_b32(rx, in ? off : kOob, 0, 0);
                } else {
                    const uint32_t lo = static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(rx, in ? off : kOob, 0, 0));
                    const uint32_t hi = static_cast<uint16_t>(__builtin_amdgcn_raw_buffer_load_b16(rx, in && c + 1 < C ? off + 2 : kOob, 0, 0));
                    d[i][u] = lo | (hi << 16);
                }
            }
        }
    };
    auto unpack = [&](uint32_t b, int q) __attribute__((always_inline)) -> float {
        if constexpr (ES == 4) return __uint_as_float(b);
        else return S::to_f32(__builtin_bit_cast(Elem, static_cast<uint16_t>(b >> (16 * q))));
    };
    // V of the loaded windows into buffer `buf`; the 16-byte pieces of a tile's
    // 64 bytes are XOR-swizzled by (tile / 4) % 4, so that a fragment read (16
    // tiles, one piece) meets every LDS bank once
    auto transform = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (i == 1 && !two) continue;
            const int tile = (tid >> 4) + 32 * i;
            const int at = tile * k1dChunk + ((((run >> 2) ^ (tile >> 2)) & 3) << 4) + (run & 3) * 4;
#pragma unroll
            for (int a = 0; a < ALPHA; ++a) {
                uint32_t bits = 0;
#pragma unroll
                for (int q = 0; q < VEC; ++q) {
                    float acc = 0.0f;
#pragma unroll
                    for (int u = 0; u < TT; ++u) acc = __builtin_fmaf(itab.bt[a * TT + u], unpack(d[i][u], q), acc);
                    if constexpr (ES == 4) bits = __float_as_uint(acc);
                    else bits |= static_cast<uint32_t>(__builtin_bit_cast(uint16_t, S::from_f32(acc))) << (16 * q);
                }
                *reinterpret_cast<uint32_t*>(&vb[buf][a * kPoint + at]) = bits;
            }
        }
    };
    // U fragments: channel row k0 + 16 wk + l16 (the last row past K, never
    // stored), 16-byte piece grp of the chunk, zero past the row
    const int kr = k0 + wk * 16 + l16 < K ? k0 + wk * 16 + l16 : K - 1;
    const uint32_t uoff = static_cast<uint32_t>(kr) * static_cast<uint32_t>(mp.rb) + grp * 16;
    u32x4 fu[ALPHA];
    auto load_u = [&](int ck) __attribute__((always_inline)) {
        const bool in = ck * k1dChunk + grp * 16 < mp.rb;
#pragma unroll
        for (int a = 0; a < ALPHA; ++a) {
            const auto ru = make_rsrc(U + static_cast<int64_t>(a) * static_cast<uint32_t>(mp.plane_u),
                                      static_cast<uint32_t>(mp.plane_u));
            fu[a] = __builtin_amdgcn_raw_buffer_load_b128(ru, in ? uoff + ck * k1dChunk : kOob, 0, 0);
        }
    };
    f32x4 acc[ALPHA][2];
#pragma unroll
    for (int a = 0; a < ALPHA; ++a)
#pragma unroll
        for (int w = 0; w < 2; ++w) acc[a][w] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const int frag = (wt * 32 + l16) * k1dChunk + (((grp ^ (l16 >> 2)) & 3) << 4);

    // U of the next chunk and the windows after it are requested as soon as
    // their registers are free, a phase before they are needed
    load_u(0);
    load(0);
    transform(0);
    if (mp.n_chunks > 1) load(1);
    __syncthreads();
    int buf = 0;
    for (int ck = 0; ck < mp.n_chunks; ++ck) {
        if constexpr (D == 0) {
            // fp32: a chunk's sum, then the chunks' (fewer roundings than one
            // chain over C); the four instructions of a sum depend on each
            // other, so the sums of a few points go side by side
            constexpr int kSide = ALPHA <= 9 ? 3 : 1;
#pragma unroll
            for (int a0 = 0; a0 < ALPHA; a0 += kSide) {
                f32x4 part[kSide][2], fv[kSide][2];
#pragma unroll
                for (int i = 0; i < kSide; ++i)
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        part[i][w] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                        if (a0 + i < ALPHA)
                            fv[i][w] = *reinterpret_cast<const f32x4*>(&vb[buf][(a0 + i) * kPoint + w * 16 * k1dChunk + frag]);
                    }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int i = 0; i < kSide; ++i)
#pragma unroll
                        for (int w = 0; w < 2; ++w)
                            if (a0 + i < ALPHA)
                                part[i][w] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(fu[a0 + i][e]), fv[i][w][e],
                                                                                  part[i][w], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < kSide; ++i)
#pragma unroll
                    for (int w = 0; w < 2; ++w)
                        if (a0 + i < ALPHA) acc[a0 + i][w] += part[i][w];
            }
        } else {
#pragma unroll
            for (int a = 0; a < ALPHA; ++a)
#pragma unroll
                for (int w = 0; w < 2; ++w) {
                    const u32x4 fv = *reinterpret_cast<const u32x4*>(&vb[buf][a * kPoint + w * 16 * k1dChunk + frag]);
                    mma_1d<D>(fu[a], fv, acc[a][w]);
                }
        }
        if (ck + 1 < mp.n_chunks) {
            load_u(ck + 1);
            transform(buf ^ 1);
            if (ck + 2 < mp.n_chunks) load(ck + 2);
        }
        __syncthreads();
        buf ^= 1;
    }
    // y[o] = sum_a A^T[o][a] M[a], a ascending: four channels of tile l16
    const int k = k0 + wk * 16 + 4 * grp;
    if (k >= K) return;
    const bool vec = (K & 3) == 0;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const int64_t t = t0 + wt * 32 + w * 16 + l16;
        if (t >= T) continue;
        const uint32_t n = fast_div(static_cast<uint32_t>(t), mp.tl);
        const int tx = static_cast<int>(static_cast<uint32_t>(t) - n * mp.tl.d);
        Elem* dst = y + (static_cast<int64_t>(n) * L + tx * MM) * K + k;
#pragma unroll
        for (int o = 0; o < MM; ++o) {
            if (tx * MM + o >= L) break;
            Elem e[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float v = 0.0f;
#pragma unroll
                for (int a = 0; a < ALPHA; ++a) v = __builtin_fmaf(otab.at[o * ALPHA + a], acc[a][w][r], v);
                e[r] = S::from_f32(v);
            }
            Elem* p = dst + static_cast<int64_t>(o) * K;
            if (vec) {
                if constexpr (ES == 4) *reinterpret_cast<u32x4*>(p) = __builtin_bit_cast(u32x4, e);
                else *reinterpret_cast<u32x2*>(p) = __builtin_bit_cast(u32x2, e);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (k + r < K) p[r] = e[r];
            }
        }
    }
}

inline unsigned blocks_1d(int64_t n) { return static_cast<unsigned>((n + kBlock1d - 1) / kBlock1d); }
inline bool grid_ok(int64_t n) { return (n + kBlock1d - 1) / kBlock1d <= 0x7fffffff; }

}  // namespace

template <int D>
hipError_t launch_kernel_transform_1d_t(const Geometry& g, const KernelTable& tab, const void* w, void* U,
                                        hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    if (g.alpha > kMaxAlpha || !grid_ok(g.K * g.Cp)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(kernel_transform_1d<Elem>, dim3(blocks_1d(g.K * g.Cp)), dim3(kBlock1d), 0, stream, tab,
                       static_cast<const Elem*>(w), static_cast<Elem*>(U), g.K, g.C, g.Cp, g.alpha);
    return hipGetLastError();
}

template <int D>
hipError_t launch_input_transform_1d_t(const Geometry& g, const InputTable& tab, const void* x, void* V,
                                       hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    if (g.alpha > kMaxAlpha || g.t > kMaxTile || !grid_ok(g.T * g.Cp)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(input_transform_1d<Elem>, dim3(blocks_1d(g.T * g.Cp)), dim3(kBlock1d), 0, stream, tab,
                       static_cast<const Elem*>(x), static_cast<Elem*>(V), g.W, g.C, g.Cp, g.tw, g.T, g.m, g.t,
                       g.alpha);
    return hipGetLastError();
}

template <int D>
hipError_t launch_output_transform_1d_t(const Geometry& g, const OutputTable& tab, const float* M, void* y,
                                        hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    if (g.alpha > kMaxAlpha || g.m > kMaxTile || !grid_ok(g.T * g.K)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(output_transform_1d<Elem>, dim3(blocks_1d(g.T * g.K)), dim3(kBlock1d), 0, stream, tab, M,
                       static_cast<Elem*>(y), g.W, g.K, g.Kp, g.tw, g.T, g.m, g.alpha);
    return hipGetLastError();
}

// The fused kernel takes the (tile, alpha') shapes of the compiled 2D transforms up to ten
// points (in fp32 thirteen took 70 against 64 us for 32x2000, 64 -> 64: the
// points' sums fill the registers), inputs within 1 GiB and planes of U within
// 32-bit offsets.
template <int D>
bool conv1d_fused_supported_t(const Geometry& g) {
    const int64_t es = D == 0 ? 4 : 2;
    return g.alpha <= k1dMaxAlpha && transform_shape_supported(g.t, g.alpha) && g.N * g.W * g.C * es <= (int64_t(1) << 30) &&
           g.T < (int64_t(1) << 30) && g.W < (int64_t(1) << 29) && g.K < (int64_t(1) << 30) &&
           g.K * g.Cp * es < 0x7fffffffLL;
}
template <int D>
bool conv1d_fused_chosen_t(const Geometry& g) {
    if (!conv1d_fused_supported_t<D>(g)) return false;
    return conv1d_one_kernel_pays(g.T, g.Cp, g.K, g.Kp, g.alpha, D == 0 ? 4 : 2);
}

template <int D>
hipError_t launch_conv1d_fused_t(const Geometry& g, const InputTable& itab, const OutputTable& otab, const void* x,
                                 const void* U, void* y, hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    if (!conv1d_fused_supported_t<D>(g)) return hipErrorInvalidValue;
    const int64_t es = sizeof(Elem);
    Map1d mp;
    mp.tl = make_fastdiv(g.tw);
    mp.xbytes = static_cast<uint32_t>(g.N * g.W * g.C * es);
    mp.kw = conv1d_waves_k(g.K);
    mp.n_kb = static_cast<int>(conv1d_k_blocks(g.K));
    mp.rb = static_cast<int>(g.Cp * es);
    mp.n_chunks = static_cast<int>(conv1d_chunks(g.Cp, es));
    mp.plane_u = static_cast<int>(g.K * g.Cp * es);
    const int64_t blocks = conv1d_blocks(g.T, g.K);
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
#define WG_1D_CASE(TT, A)                                                                                         \
    if constexpr (A <= k1dMaxAlpha)                                                                               \
    if (g.t == TT && g.alpha == A) {                                                                              \
        hipLaunchKernelGGL((conv1d_fused_kernel<D, TT, A>), dim3(static_cast<unsigned>(blocks)),                  \
                           dim3(64 * k1dWaves), 0, stream, static_cast<const Elem*>(x),                           \
                           static_cast<const unsigned char*>(U), static_cast<Elem*>(y), itab, otab, g, mp);       \
        return hipGetLastError();                                                                                 \
    }
    WG_TRANSFORM_SHAPES(WG_1D_CASE)
    WG_TRANSFORM_SHAPES_ODD(WG_1D_CASE)
#undef WG_1D_CASE
    return hipErrorInvalidValue;
}

#define WG_1D_INSTANCES(D)                                                                                       \
    template hipError_t launch_kernel_transform_1d_t<D>(const Geometry&, const KernelTable&, const void*, void*, \
                                                        hipStream_t);                                            \
    template hipError_t launch_input_transform_1d_t<D>(const Geometry&, const InputTable&, const void*, void*,   \
                                                       hipStream_t);                                             \
    template hipError_t launch_output_transform_1d_t<D>(const Geometry&, const OutputTable&, const float*,       \
                                                        void*, hipStream_t);                                     \
    template bool conv1d_fused_chosen_t<D>(const Geometry&);                                                     \
    template hipError_t launch_conv1d_fused_t<D>(const Geometry&, const InputTable&, const OutputTable&,         \
                                                 const void*, const void*, void*, hipStream_t);
WG_1D_INSTANCES(0)
WG_1D_INSTANCES(1)
WG_1D_INSTANCES(2)
#undef WG_1D_INSTANCES

}  // namespace wg
