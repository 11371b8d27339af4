// Winograd transforms of eq. (2) (Barabasz & Gregg, arXiv 1905.05233) for
// gfx950: the kernel transform U = G g G^T, the input transform V = B^T d B
// and the output transform Y = A^T M A fused with the NHWC store.
//
// All three stream channel-last data: a wavefront's loads and stores sweep
// consecutive channels of NHWC / channel-last buffers (coalesced).  The kernel
// transform runs one thread per (domain row, kernel, channels), the input
// transform one thread per (tile, channels) (input_regs.hpp), the output
// transform one thread per (tile, output channel, group of output rows)
// (output_regs.hpp) or, for layers of few such threads, one workgroup per (tile,
// 64 output channels) with its output rows split over the waves.  The transform
// matrices arrive by value
// in the kernel-argument segment (uniform across the grid, so they live in
// scalar registers); the small matrices are applied as two separable 1D passes
// in fp32 registers with ascending-index fused multiply-adds, and results are
// rounded to the storage dtype once, at the store.
//
// This file is compiled once per storage dtype (WG_DTYPE = 0 fp32, 1 fp16,
// 2 bf16); each (input tile, alpha') shape is a template instance so that the
// register arrays have compile-time sizes.
#include <algorithm>
#include <utility>

#include "coefs.hpp"
#include "device_common.hpp"
#include "input_regs.hpp"
#include "kernels.hpp"
#include "output_regs.hpp"

#ifndef WG_DTYPE
#error "compile with -DWG_DTYPE=0|1|2"
#endif

namespace wg {

namespace {

constexpr int kBlock = 256;

// ----------------------------------------------------------------- kernel
// U[xi = a*alpha + b][k][c] = sum_j (sum_i G[a][i] g[i][j]) G[b][j]; one thread
// per (row a, k, run of kRun channels), runs fastest, so loads and stores are
// kRun elements per lane (16 bytes in the stand-alone kernel; 4 channels when
// it shares a launch with the input transform, to keep that kernel's register
// count low).  kWhole: C is a multiple of the run, so the runs of w are
// aligned; otherwise w is read element by element.
constexpr int64_t kKtThreads = int64_t(1) << 15;
template <int BYTES> struct RunBits;
template <> struct RunBits<16> { using type = uint4; };
template <> struct RunBits<8> { using type = uint2; };

// Divisors of the kernel transform's thread ids: runs per row of C, kernels.
// 32-bit arithmetic where the launch's ids fit (64-bit divisions cost more than
// the transform's own arithmetic).
struct KernelMap {
    FastDiv runs, k;
    int small;   // ids below 2^31
};
inline KernelMap make_kernel_map(const Geometry& g, int run, int64_t threads) {
    KernelMap mp;
    mp.runs = make_fastdiv(g.Cp / run);
    mp.k = make_fastdiv(g.K);
    mp.small = threads < (int64_t(1) << 31) ? 1 : 0;
    return mp;
}
// gid = (row K + k) runs + c / kRun
__device__ __forceinline__ void kernel_map_split(const KernelMap& mp, int64_t gid, int64_t& c_run, int64_t& k, int64_t& row) {
    if (mp.small) {
        const uint32_t i = static_cast<uint32_t>(gid), kr = fast_div(i, mp.runs), r = fast_div(kr, mp.k);
        c_run = i - kr * mp.runs.d;
        k = kr - r * mp.k.d;
        row = r;
    } else {
        c_run = gid % mp.runs.d;
        k = gid / mp.runs.d % mp.k.d;
        row = gid / mp.runs.d / mp.k.d;
    }
}

template <typename Elem, int ALPHA, int kRun, bool kWhole>
__device__ __forceinline__ void kernel_transform_run(const KernelTable& tab, const Elem* __restrict__ w,
                                                     Elem* __restrict__ U, int64_t K, int64_t C, int64_t Cp,
                                                     const KernelMap& mp, int64_t gid) {
    using S = Storage<Elem>;
    using Bits = typename RunBits<kRun * sizeof(Elem)>::type;
    if (gid >= ALPHA * K * mp.runs.d) return;
    int64_t c, k, row;
    kernel_map_split(mp, gid, c, k, row);
    c *= kRun;
    const int a = static_cast<int>(row);
    const int64_t plane = K * Cp;
    float g[3][3][kRun];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const Elem* src = w + ((k * 3 + i) * 3 + j) * C + c;
            Elem e[kRun];
            if constexpr (kWhole) {
                // a run starts inside C only if it ends inside it (for fp32, Cp may exceed C by a run)
                *reinterpret_cast<Bits*>(e) = c < C ? *reinterpret_cast<const Bits*>(src) : Bits{};
            } else {
#pragma unroll
                for (int q = 0; q < kRun; ++q) e[q] = c + q < C ? src[q] : S::from_f32(0.0f);
            }
#pragma unroll
            for (int q = 0; q < kRun; ++q) g[i][j][q] = S::to_f32(e[q]);
        }
    float Gg[3][kRun];
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
        for (int q = 0; q < kRun; ++q) {
            float acc = 0.0f;
#pragma unroll
            for (int i = 0; i < 3; ++i) acc = __builtin_fmaf(tab.g[a * 3 + i], g[i][j][q], acc);
            Gg[j][q] = acc;
        }
    Elem* out = U + static_cast<int64_t>(a) * ALPHA * plane + k * Cp + c;
#pragma unroll
    for (int b = 0; b < ALPHA; ++b) {
        Elem e[kRun];
#pragma unroll
        for (int q = 0; q < kRun; ++q) {
            float acc = 0.0f;
#pragma unroll
            for (int j = 0; j < 3; ++j) acc = __builtin_fmaf(Gg[j][q], tab.g[b * 3 + j], acc);
            e[q] = S::from_f32(acc);   // channels past C: g = 0, so zeros
        }
        *reinterpret_cast<Bits*>(out + b * plane) = *reinterpret_cast<const Bits*>(e);
    }
}

// The same, one thread per (k, run of kRun channels) computing every row a:
// the 3x3 taps are loaded once instead of once per row, and a launch needs
// alpha' times fewer threads (the form the combined kernel/input launch uses,
// so that fewer kernel-transform workgroups precede the input-transform ones).
// Each output is computed in the same order as above.
template <typename Elem, int ALPHA, int kRun, bool kWhole>
__device__ __forceinline__ void kernel_transform_rows(const KernelTable& tab, const Elem* __restrict__ w,
                                                      Elem* __restrict__ U, int64_t K, int64_t C, int64_t Cp,
                                                      const KernelMap& mp, int64_t gid) {
    using S = Storage<Elem>;
    using Bits = typename RunBits<kRun * sizeof(Elem)>::type;
    if (gid >= K * mp.runs.d) return;
    int64_t c, k, row;
    kernel_map_split(mp, gid, c, k, row);
    c *= kRun;
    const int64_t plane = K * Cp;
    float g[3][3][kRun];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const Elem* src = w + ((k * 3 + i) * 3 + j) * C + c;
            Elem e[kRun];
            if constexpr (kWhole) {
                *reinterpret_cast<Bits*>(e) = c < C ? *reinterpret_cast<const Bits*>(src) : Bits{};
            } else {
#pragma unroll
                for (int q = 0; q < kRun; ++q) e[q] = c + q < C ? src[q] : S::from_f32(0.0f);
            }
#pragma unroll
            for (int q = 0; q < kRun; ++q) g[i][j][q] = S::to_f32(e[q]);
        }
    Elem* out = U + k * Cp + c;
#pragma unroll
    for (int a = 0; a < ALPHA; ++a) {
        float Gg[3][kRun];
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int q = 0; q < kRun; ++q) {
                float acc = 0.0f;
#pragma unroll
                for (int i = 0; i < 3; ++i) acc = __builtin_fmaf(tab.g[a * 3 + i], g[i][j][q], acc);
                Gg[j][q] = acc;
            }
#pragma unroll
        for (int b = 0; b < ALPHA; ++b) {
            Elem e[kRun];
#pragma unroll
            for (int q = 0; q < kRun; ++q) {
                float acc = 0.0f;
#pragma unroll
                for (int j = 0; j < 3; ++j) acc = __builtin_fmaf(Gg[j][q], tab.g[b * 3 + j], acc);
                e[q] = S::from_f32(acc);
            }
            *reinterpret_cast<Bits*>(out + (a * ALPHA + b) * plane) = *reinterpret_cast<const Bits*>(e);
        }
    }
}

template <typename Elem, int ALPHA, bool kWhole>
__global__ __launch_bounds__(kBlock) void kernel_transform(KernelTable tab, const Elem* __restrict__ w,
                                                           Elem* __restrict__ U, int64_t K, int64_t C,
                                                           int64_t Cp, KernelMap mp) {
    kernel_transform_run<Elem, ALPHA, 16 / sizeof(Elem), kWhole>(tab, w, U, K, C, Cp, mp,
                                                                 static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x);
}

// ------------------------------------------------------------------ input
// The input transform itself is in input_regs.hpp.

// Channels per thread: pairs (4-byte accesses) in 16-bit storage where the
// window's registers allow it, C is even, so that no run straddles two pixels,
// and the layer has threads enough (kInFirstUnits).  With windows read from HBM pairs measured 53 against 57 us for
// 32x56x56x256; from 8x8 windows on their registers halve the waves in flight
// (9.2 against 8.2 us for 16x28x28x256, alpha' = 10).
template <typename Elem> constexpr bool input_pairs(int tt) { return sizeof(Elem) == 2 && tt <= 6; }
// Row groups: large windows of small layers split the domain rows over four
// workgroups' threads, each computing a quarter of V's rows from its own copy of
// the window.  It pays while the layer has too few threads to occupy the
// SIMDs: 4x56x56x64 in fp32 with 8x8 tiles (12.5 thousand threads) 10.6 -> 6.8
// us, while 16x28x28x256 with 6x6 tiles (102 thousand) went from 8.1 to 9.4 us.
//
// Windows of 12 and more with alpha' over 12, and 10x10 ones with alpha' = 12,
// split at every size: with all rows in one thread the coefficients overflow the
// scalar registers, and the code (60 KB for the latter, 120 - 266 KB for the
// others) the instruction cache; a group's part of it fits.  221 thousand threads
// in bf16, all rows -> split: t = 10, alpha' = 12 64 -> 39 us; 12, 13 126 -> 84;
// 12, 15 164 -> 87; 14, 14 285 -> 103; 14, 16 334 -> 139.  The others have at most
// 39 KB, and lose: 12x12 with alpha' = 12 49 -> 55, 10x10 with alpha' = 13 41 -> 64.
//
// 14x14 windows in 16 bits take two rows a group up to alpha' = 15: with four the
// window and the rows' sums need 320 registers, one wave per SIMD (221 thousand
// threads, alpha' = 14: four rows 132 us, two 103; alpha' = 16: 139 and 145).  Those
// and the fp32 ones come within a few registers of two waves per SIMD, so they are
// held to it.
constexpr int kInGroups = 4;
constexpr int input_groups(int tt, int alpha, int es) {
    return tt >= 14 && es == 2 && alpha <= 15 ? (alpha + 1) / 2 : tt >= 8 ? kInGroups : 1;
}
constexpr bool input_always_split(int tt, int alpha) { return tt >= 12 ? alpha > 12 : tt == 10 && alpha == 12; }
constexpr int input_waves(int tt, int groups, int es) { return tt >= 14 && (es == 4 || groups > kInGroups) ? 2 : 1; }
constexpr int64_t kInFewThreads = int64_t(1) << 15;
// Layers of at most one workgroup of one-channel threads per CU are bound by one
// thread's latency: they take one channel per thread, and in the joint launch
// their units go ahead of the kernel transform, so that they don't start last.
// The joint launch, F(4x4) with a^2+1 in bf16, pairs behind the kernel transform
// -> pairs ahead -> single channels ahead: 1x14x14, 512 -> 512 7.71 -> 7.33 -> 7.07 us,
// 1x28x28, 256 -> 256 5.15 -> 4.99 -> 4.33, 4x14x14, 512 -> 32 4.79 -> 4.42 -> 3.74.
// With more units the short kernel transform stays ahead.
constexpr int64_t kInFirstUnits = 256;

template <typename Elem, int TT, int ALPHA, class CO, int VEC, int RG, InputPart PART, bool RELU>
__global__ __launch_bounds__(kInBlock, (input_waves(TT, RG, sizeof(Elem)))) void input_transform(InputTable tab, const Elem* __restrict__ x,
                                                            unsigned char* __restrict__ V, Geometry geo, InputMap mp) {
    input_regs_unit<Elem, TT, ALPHA, CO, VEC, RG, PART, RELU>(tab, x, V, geo, mp, blockIdx.x, gridDim.x);
}

// The kernel and input transforms are independent: conv2d runs them as one
// launch.  n_kt workgroups run the kernel transform, the rest are
// input-transform units (one launch instead of two, and the short kernel
// transform overlaps the input transform); n_first units (all or none) go
// ahead of the kernel transform.  kt_rows: one kernel-transform
// thread per (k, 4-channel run) for every row a, else one per row; whole: C is a
// multiple of 16 bytes, so the runs of w are aligned.
template <typename Elem, int TT, int ALPHA, class CO, int VEC, int RG, bool RELU>
__global__ __launch_bounds__(kInBlock) void kernel_input_transform(
    KernelTable ktab, InputTable itab, const Elem* __restrict__ w, const Elem* __restrict__ x,
    Elem* __restrict__ U, unsigned char* __restrict__ V, Geometry geo, InputMap mp, KernelMap kmp, int64_t n_kt, int64_t n_first,
    int kt_rows, int whole) {
    const int64_t bid = blockIdx.x;
    if (bid >= n_first && bid < n_first + n_kt) {
        const int64_t gid = (bid - n_first) * kInBlock + threadIdx.x;
        if (kt_rows && whole) kernel_transform_rows<Elem, ALPHA, 4, true>(ktab, w, U, geo.K, geo.C, geo.Cp, kmp, gid);
        else if (kt_rows) kernel_transform_rows<Elem, ALPHA, 4, false>(ktab, w, U, geo.K, geo.C, geo.Cp, kmp, gid);
        else if (whole) kernel_transform_run<Elem, ALPHA, 4, true>(ktab, w, U, geo.K, geo.C, geo.Cp, kmp, gid);
        else kernel_transform_run<Elem, ALPHA, 4, false>(ktab, w, U, geo.K, geo.C, geo.Cp, kmp, gid);
        return;
    }
    input_regs_unit<Elem, TT, ALPHA, CO, VEC, RG, kInTop, RELU>(itab, x, V, geo, mp, bid < n_first ? bid : bid - n_kt, gridDim.x - n_kt);
}

// ----------------------------------------------------------------- output
// y[n][ty*m+o][tx*m+p][k] = sum_b (sum_a A^T[o][a] M[a][b]) A^T[p][b]
//
// For layers of few threads (others: output_regs.hpp).  One workgroup per (tile,
// 64 output channels); the m output rows are split
// over its waves (wave g computes rows [g*R, g*R + R) for its 64 channels).
// Every wave loads the tile's alpha'^2 values of M for its channels, all
// before any arithmetic (coalesced 256-byte rows; the repeats across the
// workgroup's waves are served by the caches), then runs pass 1 in ascending
// a and pass 2 in ascending b and stores its rows, masked at the right and
// bottom edges of the image.
constexpr int kOutCh = 64;   // output channels per workgroup, one per lane

// rows per wave: the split that measured fastest
constexpr int output_rows_per_wave(int alpha) { return alpha >= 9 ? 3 : 2; }

// (tile, output channel) pairs from which the form of output_regs.hpp is taken: it
// has fewer waves, which layers of fewer pairs need to hide the loads of M
// (1x14x14x512 in bf16 has 8 thousand; 6x75x91x120 in fp16, 315 thousand, 17.4 us
// here and 12.3 there; 32x28x28x512 28.0 and 26.7).
constexpr int64_t kOutManyThreads = int64_t(1) << 17;
// Bytes of M up to which 2x2 tiles take two row groups as well, one row each: the
// second group's reads hit the 256 MB last-level cache.  alpha' = 5 in bf16, two
// groups and one: 32x28x28x256 (161 MB) 24.5 and 25.9 us, 4x112x112x256 (321 MB) 70.9
// and 65.2.  Larger tiles read M twice for half of their rows each.
constexpr int64_t kOutCachedBytes = int64_t(256) << 20;

template <int MM, int ALPHA>
struct OutputShape {
    static constexpr int kR = output_rows_per_wave(ALPHA);
    static constexpr int kG = (MM + kR - 1) / kR;   // waves (row groups)
    static constexpr int kThreads = 64 * kG;
};

template <typename Elem, int MM, int ALPHA, int O0, class CO>
__device__ __forceinline__ void output_rows(const OutputTable& tab, const float* __restrict__ in, int64_t plane,
                                            Elem* __restrict__ yk, int64_t hr0, int64_t wc0, const Geometry& geo) {
    using S = Storage<Elem>;
    constexpr int R = OutputShape<MM, ALPHA>::kR;
    float Mv[ALPHA][ALPHA];
#pragma unroll
    for (int a = 0; a < ALPHA; ++a)
#pragma unroll
        for (int b = 0; b < ALPHA; ++b) Mv[a][b] = in[(a * ALPHA + b) * plane];
    // pass 1, one domain column at a time: Z[r][b] = sum_a A^T[O0+r][a] M[a][b]
    float Z[R][ALPHA];
#pragma unroll
    for (int b = 0; b < ALPHA; ++b)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float acc = 0.0f;
            if (O0 + r < MM) {
#pragma unroll
                for (int a = 0; a < ALPHA; ++a) acc = term<CO>(CO::at(tab, (O0 + r) * ALPHA + a), Mv[a][b], acc);
            }
            Z[r][b] = acc;
        }
    // pass 2 and the masked NHWC store
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t hr = hr0 + O0 + r;
        if (O0 + r >= MM || hr >= geo.H) break;
#pragma unroll
        for (int p = 0; p < MM; ++p) {
            const int64_t wc = wc0 + p;
            float acc = 0.0f;
#pragma unroll
            for (int b = 0; b < ALPHA; ++b) acc = term<CO>(CO::at(tab, p * ALPHA + b), Z[r][b], acc);
            if (wc < geo.W) yk[(hr * geo.W + wc) * geo.K] = S::from_f32(acc);
        }
    }
}

template <typename Elem, int MM, int ALPHA, class CO, int... Gs>
__device__ __forceinline__ void output_row_groups(int g, const OutputTable& tab, const float* in, int64_t plane,
                                                  Elem* yk, int64_t hr0, int64_t wc0, const Geometry& geo,
                                                  std::integer_sequence<int, Gs...>) {
    ((g == Gs ? (output_rows<Elem, MM, ALPHA, Gs * OutputShape<MM, ALPHA>::kR, CO>(tab, in, plane, yk, hr0, wc0, geo),
                 0)
              : 0),
     ...);
}

template <typename Elem, int MM, int ALPHA, class CO>
__global__ __launch_bounds__((OutputShape<MM, ALPHA>::kThreads)) void output_transform(
    OutputTable tab, const float* __restrict__ Mx, Elem* __restrict__ y, Geometry geo) {
    const int64_t nkc = (geo.K + kOutCh - 1) / kOutCh;
    const int64_t unit = blockIdx.x;
    const int64_t tile = unit / nkc;
    const int64_t k = (unit % nkc) * kOutCh + threadIdx.x % kOutCh;
    const int g = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kOutCh);
    if (k >= geo.K) return;
    const int64_t tx = tile % geo.tw;
    const int64_t ty = (tile / geo.tw) % geo.th;
    const int64_t n = tile / (geo.tw * geo.th);
    output_row_groups<Elem, MM, ALPHA, CO>(g, tab, Mx + tile * geo.Kp + k, geo.T * geo.Kp,
                                       y + n * geo.H * geo.W * geo.K + k, ty * MM, tx * MM, geo,
                                       std::make_integer_sequence<int, OutputShape<MM, ALPHA>::kG>{});
}

inline unsigned blocks_for(int64_t n) { return static_cast<unsigned>((n + kBlock - 1) / kBlock); }

}  // namespace

// ------------------------------------------------------------- launchers

template <int D>
hipError_t launch_kernel_transform_t(const Geometry& g, const KernelTable& tab, const void* w, void* U,
                                     hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    const auto* wp = static_cast<const Elem*>(w);
    auto* up = static_cast<Elem*>(U);
    constexpr int kRun = 16 / static_cast<int>(sizeof(Elem));
    const int64_t threads = static_cast<int64_t>(g.alpha) * g.K * (g.Cp / kRun);
    const unsigned nb = blocks_for(threads);
    const KernelMap mp = make_kernel_map(g, kRun, threads);
    const bool whole = g.C % kRun == 0;
    switch (g.alpha) {
#define WG_KT_CASE(A)                                                                                   \
    case A:                                                                                             \
        if (whole)                                                                                      \
            hipLaunchKernelGGL((kernel_transform<Elem, A, true>), dim3(nb), dim3(kBlock), 0, stream, tab, wp, up, \
                               g.K, g.C, g.Cp, mp);                                                       \
        else                                                                                            \
            hipLaunchKernelGGL((kernel_transform<Elem, A, false>), dim3(nb), dim3(kBlock), 0, stream, tab, wp, up, \
                               g.K, g.C, g.Cp, mp);                                                       \
        break;
        WG_KT_CASE(4) WG_KT_CASE(5) WG_KT_CASE(6) WG_KT_CASE(7) WG_KT_CASE(8) WG_KT_CASE(9)
        WG_KT_CASE(10) WG_KT_CASE(11) WG_KT_CASE(12) WG_KT_CASE(13) WG_KT_CASE(14) WG_KT_CASE(15)
        WG_KT_CASE(16)
#undef WG_KT_CASE
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// One launch of each kernel shape, with the coefficient source CO.  The images
// go in groups, and an image over 1 GiB in bands of tile rows, whose bytes and
// threads fit 32-bit arithmetic; with ktab the first launch carries the kernel
// transform.  RELU: of ReLU(x) (images of at most kInMaxBytes).
//
// Bands, and not one launch with 64-bit addresses: 1x8192x8192x64 in bf16 with
// alpha' = 7 (8.6 GB of x) 16.3 ms so with one channel per thread, 7.1 ms in
// bands of pairs.  Only images whose tile rows are too large for a band each
// are left to 64-bit addresses.
template <typename Elem, int TT, int A, class CO, bool RELU = false>
hipError_t launch_in(const Geometry& g, const KernelTable* ktab, const InputTable& tab, const Elem* wp, const Elem* xp,
                     Elem* up, Elem* vp, hipStream_t stream) {
    constexpr int ES = static_cast<int>(sizeof(Elem));
    constexpr int kM = TT - 2;
    constexpr bool kPairs = input_pairs<Elem>(TT);
    constexpr int kRG = input_groups(TT, A, ES);
    constexpr int kBigRG = input_always_split(TT, A) ? kRG : 1;   // row groups of layers of any size
    const bool few = g.T * g.Cp <= kInFirstUnits * kInBlock;
    const bool pairs = kPairs && g.C % 2 == 0 && !few;
    const int vec = pairs ? 2 : 1;
    const int64_t tiles_img = g.th * g.tw, thr_row = g.tw * (g.Cp / vec), row = g.W * g.C, x_img = g.H * row;
    InputMap mp;
    mp.per_tile = make_fastdiv(g.Cp / vec);
    mp.tw = make_fastdiv(g.tw);
    mp.plane = g.T * g.Cp * ES;
    const InputSplit sp = input_split(g.H, row * ES, g.th, thr_row, kM, kBigRG);
    if (sp.rows == 0) {
        // rows of over kInMaxBytes / t: the kernel transform apart, 64-bit addresses
        if constexpr (RELU) {
            return hipErrorInvalidValue;
        } else {
            mp.th = make_fastdiv(g.th);
            mp.threads = g.T * (g.Cp / vec);
            mp.xbytes = 0;
            const int64_t blocks = input_blocks(mp.threads, kBigRG);
            if (blocks * kInBlock > kMaxWorkItems) return hipErrorInvalidValue;
            if (ktab) {
                constexpr int D = sizeof(Elem) == 4 ? 0 : __is_same(Elem, bf16_t) ? 2 : 1;
                const hipError_t e = launch_kernel_transform_t<D>(g, *ktab, wp, up, stream);
                if (e != hipSuccess) return e;
            }
#define WG_IT_BIG(VEC)                                                                                             \
    hipLaunchKernelGGL((input_transform<Elem, TT, A, CO, VEC, kBigRG, kInFar, false>), dim3(static_cast<unsigned>(blocks)), \
                       dim3(kInBlock), 0, stream, tab, xp, reinterpret_cast<unsigned char*>(vp), g, mp)
            if constexpr (kPairs) {
                if (pairs) WG_IT_BIG(2);
                else WG_IT_BIG(1);
            } else {
                WG_IT_BIG(1);
            }
#undef WG_IT_BIG
            return hipGetLastError();
        }
    }
    // whole images (one band each, every row of it) or bands of one image
    const bool whole_images = sp.rows == g.th;
    for (int64_t n0 = 0, r0 = 0; n0 < g.N;) {
        const int64_t nn = std::min<int64_t>(sp.images, g.N - n0), nr = std::min<int64_t>(sp.rows, g.th - r0);
        const InputBand band = whole_images ? InputBand{0, g.H} : input_band(g.H, r0, nr, kM);
        const bool first = n0 == 0 && r0 == 0;
        mp.th = make_fastdiv(nr);
        mp.threads = nn * nr * thr_row;
        Geometry part = g;
        part.H = band.end - band.first;
        mp.xbytes = static_cast<uint32_t>(nn * part.H * row * ES);
        const Elem* xs = xp + n0 * x_img + band.first * row;
        auto* vs = reinterpret_cast<unsigned char*>(vp) + (n0 * tiles_img + r0 * g.tw) * g.Cp * ES;
        const bool split = kBigRG > 1 || (kRG > 1 && mp.threads <= kInFewThreads);
        const int64_t units = input_blocks(mp.threads, split ? kRG : 1);
        if (ktab && first) {
            // the kernel transform's workgroups, a multiple of 8, so the input
            // transform's ids keep their XCD (id mod 8).  One thread for every
            // row a of a (k, 4-channel run) loads the taps once, but needs
            // kKtThreads of them to cover the latency of its stores: alpha' = 7
            // in bf16 with next to no input, K x C = 256 x 256 (16 thousand
            // threads) 5.2 us against 4.8 with a thread per row, 512 x 256 5.8
            // against 6.1, 500 x 512 6.8 against 8.7.
            const int64_t kt_runs = g.K * (g.Cp / 4);
            const int kt_rows = kt_runs >= kKtThreads ? 1 : 0;
            const int64_t kt_thr = kt_rows ? kt_runs : kt_runs * A;
            const KernelMap kmp = make_kernel_map(g, 4, kt_thr);
            const int64_t n_kt = (kt_thr + 8 * kInBlock - 1) / (8 * kInBlock) * 8;
            if (n_kt + units > 0x7fffffff) return hipErrorInvalidValue;
            const dim3 grid(static_cast<unsigned>(n_kt + units));
            const int64_t n_first = few ? units : 0;
            const int whole = g.C % (16 / ES) == 0 ? 1 : 0;
#define WG_KIT(VEC, RG)                                                                                           \
    hipLaunchKernelGGL((kernel_input_transform<Elem, TT, A, CO, VEC, RG, RELU>), grid, dim3(kInBlock), 0, stream, *ktab, \
                       tab, wp, xs, up, vs, part, mp, kmp, n_kt, n_first, kt_rows, whole)
            if constexpr (kPairs) {
                if (pairs) WG_KIT(2, 1);
                else WG_KIT(1, 1);
            } else if constexpr (TT <= 8) {
                if (split) WG_KIT(1, kRG);
                else WG_KIT(1, 1);
            }
#undef WG_KIT
        } else {
            if (units > 0x7fffffff) return hipErrorInvalidValue;
            const dim3 grid(static_cast<unsigned>(units));
#define WG_IT(VEC, RG)                                                                                             \
    do {                                                                                                           \
        if (r0 == 0)                                                                                               \
            hipLaunchKernelGGL((input_transform<Elem, TT, A, CO, VEC, RG, kInTop, RELU>), grid, dim3(kInBlock), 0, \
                               stream, tab, xs, vs, part, mp);                                                     \
        else if constexpr (!RELU)                                                                                  \
            hipLaunchKernelGGL((input_transform<Elem, TT, A, CO, VEC, RG, kInBelow, false>), grid, dim3(kInBlock), \
                               0, stream, tab, xs, vs, part, mp);                                                  \
    } while (0)
            if constexpr (kPairs) {
                if (pairs) WG_IT(2, 1);
                else WG_IT(1, 1);
            } else {
                if (split) WG_IT(1, kRG);
                else WG_IT(1, kBigRG);
            }
#undef WG_IT
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        r0 += nr;
        if (r0 == g.th) {
            r0 = 0;
            n0 += nn;
        }
    }
    return hipSuccess;
}

template <typename Elem, int TT, int A, class CO, int G>
hipError_t launch_ot_regs(const Geometry& g, const OutputTable& tab, const float* M, Elem* yp, hipStream_t stream) {
    // launches of whole tiles (one but for huge layers)
    OutputMap mp;
    mp.per_tile = make_fastdiv(g.K);
    mp.tw = make_fastdiv(g.tw);
    mp.th = make_fastdiv(g.th);
    const int64_t per = output_tiles_per_launch(g.K, G);
    for (int64_t t0 = 0; t0 < g.T; t0 += per) {
        mp.tile0 = t0;
        mp.threads = std::min<int64_t>(per, g.T - t0) * g.K;
        hipLaunchKernelGGL((output_transform_regs<Elem, TT - 2, A, CO, G>),
                           dim3(static_cast<unsigned>(output_blocks(mp.threads, G))), dim3(kOutBlock), 0, stream, tab, M, yp, g, mp);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename Elem, int TT, int A, class CO>
hipError_t launch_ot(const Geometry& g, const OutputTable& tab, const float* M, Elem* yp, hipStream_t stream) {
    if (g.T * g.K >= kOutManyThreads && g.T < (int64_t(1) << 31) && g.K <= output_max_pairs(kOutGroups)) {
        if constexpr (TT == 4)
            if (int64_t(A) * A * g.T * g.Kp * 4 > kOutCachedBytes) return launch_ot_regs<Elem, TT, A, CO, 1>(g, tab, M, yp, stream);
        return launch_ot_regs<Elem, TT, A, CO, kOutGroups>(g, tab, M, yp, stream);
    }
    const int64_t units = g.T * ((g.K + kOutCh - 1) / kOutCh);
    if (units > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL((output_transform<Elem, TT - 2, A, CO>), dim3(static_cast<unsigned>(units)),
                       dim3(OutputShape<TT - 2, A>::kThreads), 0, stream, tab, M, yp, g);
    return hipGetLastError();
}

// Dispatch: the constant-coefficient instance of a built-in plan (builtin =
// its id, when the shape matches), else the kernel-argument tables.
template <int D>
bool input_relu_supported_t(const Geometry& g, int builtin) {
    return builtin >= 0 && g.t <= 8 && g.H * g.W * g.C * dtype_bytes(D) <= kInMaxBytes &&
           g.th * g.tw * g.Cp <= 0x7fffffff;
}

template <int D>
hipError_t launch_input_transform_t(const Geometry& g, const InputTable& tab, const void* x, void* V,
                                    int builtin, bool relu, hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    const auto* xp = static_cast<const Elem*>(x);
    auto* vp = static_cast<Elem*>(V);
    if (relu && !input_relu_supported_t<D>(g, builtin)) return hipErrorInvalidValue;
    if (relu) {
        switch (builtin) {
#define WG_IT_RELU(ID, TT, A)                                                                              \
    case ID:                                                                                               \
        return launch_in<Elem, TT, A, ConstCoefs<BuiltinPlan##ID>, true>(g, nullptr, tab, nullptr, xp, nullptr, vp, stream);
            WG_BUILTIN_PLANS(WG_IT_RELU)
#undef WG_IT_RELU
            default:
                return hipErrorInvalidValue;
        }
    }
    switch (builtin) {
#define WG_IT_BUILTIN(ID, TT, A)                                                                           \
    case ID:                                                                                               \
        if (g.t == TT && g.alpha == A) \
            return launch_in<Elem, TT, A, ConstCoefs<BuiltinPlan##ID>>(g, nullptr, tab, nullptr, xp, nullptr, vp, stream); \
        break;
        WG_BUILTIN_PLANS(WG_IT_BUILTIN)
#undef WG_IT_BUILTIN
        default:
            break;
    }
#define WG_IT_CASE(TT, A) \
    if (g.t == TT && g.alpha == A) \
        return launch_in<Elem, TT, A, RuntimeCoefs>(g, nullptr, tab, nullptr, xp, nullptr, vp, stream);
    WG_TRANSFORM_SHAPES(WG_IT_CASE)
    WG_TRANSFORM_SHAPES_ODD(WG_IT_CASE)
#undef WG_IT_CASE
    return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_kernel_input_transform_t(const Geometry& g, const KernelTable& ktab, const InputTable& itab,
                                           const void* w, const void* x, void* U, void* V, int builtin, bool relu,
                                           hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    const auto* wp = static_cast<const Elem*>(w);
    const auto* xp = static_cast<const Elem*>(x);
    auto* up = static_cast<Elem*>(U);
    auto* vp = static_cast<Elem*>(V);
    if (g.t > 8) {   // larger tiles: two launches (a combined kernel is large and saves little)
        const hipError_t e = launch_kernel_transform_t<D>(g, ktab, w, U, stream);
        return e != hipSuccess ? e : launch_input_transform_t<D>(g, itab, x, V, builtin, relu, stream);
    }
    if (relu && !input_relu_supported_t<D>(g, builtin)) return hipErrorInvalidValue;
    if (relu) {
        switch (builtin) {
#define WG_KIT_RELU(ID, TT, A)                                                                             \
    case ID:                                                                                               \
        return launch_in<Elem, TT, A, ConstCoefs<BuiltinPlan##ID>, true>(g, &ktab, itab, wp, xp, up, vp, stream);
            WG_BUILTIN_PLANS(WG_KIT_RELU)
#undef WG_KIT_RELU
            default:
                return hipErrorInvalidValue;
        }
    }
    switch (builtin) {
#define WG_KIT_BUILTIN(ID, TT, A)                                                                          \
    case ID:                                                                                               \
        if (g.t == TT && g.alpha == A)                                                                     \
            return launch_in<Elem, TT, A, ConstCoefs<BuiltinPlan##ID>>(g, &ktab, itab, wp, xp, up, vp, stream); \
        break;
        WG_BUILTIN_PLANS(WG_KIT_BUILTIN)
#undef WG_KIT_BUILTIN
        default:
            break;
    }
#define WG_KIT_CASE(TT, A)                                                                                 \
    if constexpr (TT <= 8)                                                                                 \
        if (g.t == TT && g.alpha == A)                                                                     \
            return launch_in<Elem, TT, A, RuntimeCoefs>(g, &ktab, itab, wp, xp, up, vp, stream);
    WG_TRANSFORM_SHAPES(WG_KIT_CASE)
    WG_TRANSFORM_SHAPES_ODD(WG_KIT_CASE)
#undef WG_KIT_CASE
    return hipErrorInvalidValue;
}

template <int D>
hipError_t launch_output_transform_t(const Geometry& g, const OutputTable& tab, const float* M, void* y,
                                     int builtin, hipStream_t stream) {
    using Elem = typename DTypeOf<D>::type;
    auto* yp = static_cast<Elem*>(y);
    switch (builtin) {
#define WG_OT_BUILTIN(ID, TT, A)                                                                           \
    case ID:                                                                                               \
        if (g.t == TT && g.alpha == A) return launch_ot<Elem, TT, A, ConstCoefs<BuiltinPlan##ID>>(g, tab, M, yp, stream); \
        break;
        WG_BUILTIN_PLANS(WG_OT_BUILTIN)
#undef WG_OT_BUILTIN
        default:
            break;
    }
#define WG_OT_CASE(TT, A) \
    if (g.t == TT && g.alpha == A) return launch_ot<Elem, TT, A, RuntimeCoefs>(g, tab, M, yp, stream);
    WG_TRANSFORM_SHAPES(WG_OT_CASE)
    WG_TRANSFORM_SHAPES_ODD(WG_OT_CASE)
#undef WG_OT_CASE
    return hipErrorInvalidValue;
}

template hipError_t launch_kernel_transform_t<WG_DTYPE>(const Geometry&, const KernelTable&, const void*, void*,
                                                        hipStream_t);
template bool input_relu_supported_t<WG_DTYPE>(const Geometry&, int);
template hipError_t launch_input_transform_t<WG_DTYPE>(const Geometry&, const InputTable&, const void*, void*, int,
                                                       bool, hipStream_t);
template hipError_t launch_kernel_input_transform_t<WG_DTYPE>(const Geometry&, const KernelTable&,
                                                              const InputTable&, const void*, const void*, void*,
                                                              void*, int, bool, hipStream_t);
template hipError_t launch_output_transform_t<WG_DTYPE>(const Geometry&, const OutputTable&, const float*, void*,
                                                        int, hipStream_t);

}  // namespace wg
