// Output transform Y = A^T M A of eq. (2) (Barabasz & Gregg, arXiv 1905.05233)
// in registers: one thread per (tile, output channel, group of output rows),
// fused with the masked NHWC store.
//
// y[n][ty*m+o][tx*m+p][k] = sum_b (sum_a A^T[o][a] M[a][b]) A^T[p][b], a and b
// ascending, fp32 fused multiply-adds from zero, rounded once at the store.  A
// domain column at a time: its alpha' values of M are loaded, folded into Z[o]
// and those into the m x m outputs.
//
// What bounds it: alpha'^2 / m^2 times the fp32 bytes of the output are read.  A
// workgroup's threads span consecutive (tile, channel) pairs, so none is idle
// where K is not a multiple of 64, and two row groups read M twice (the second
// time from the caches) instead of once per wave of up to four.  Against one
// workgroup per (tile, 64 channels): 6x75x91x120 in fp16 17.4 -> 12.3 us,
// 32x28x28x512 in bf16 28.0 -> 26.7 us (157 MB of M, 5.9 TB/s), 16x60x60x128 with
// 10x10 windows in fp32 42.6 -> 25.3 us.
#pragma once

#include "coefs.hpp"
#include "device_common.hpp"
#include "kernels.hpp"
#include "launch_split.hpp"

namespace wg {

struct OutputMap {
    FastDiv per_tile, tw, th;   // divisors: threads per tile, tiles per row, tile rows
    int64_t threads;            // (tile, channel) pairs of this launch (at most output_max_pairs)
    int64_t tile0;              // its first tile
};

template <typename Elem, int MM, int ALPHA, class CO, int O0, int O1>
__device__ __forceinline__ void output_regs_rows(const OutputTable& tab, const float* __restrict__ in, int64_t plane,
                                                 Elem* __restrict__ yk, int64_t hr0, int64_t wc0, const Geometry& geo) {
    using S = Storage<Elem>;
    constexpr int NR = O1 - O0;
    float Y[NR][MM];
#pragma unroll
    for (int o = 0; o < NR; ++o)
#pragma unroll
        for (int p = 0; p < MM; ++p) Y[o][p] = 0.0f;
#pragma unroll
    for (int b = 0; b < ALPHA; ++b) {
        float col[ALPHA];
#pragma unroll
        for (int a = 0; a < ALPHA; ++a) col[a] = in[(a * ALPHA + b) * plane];
#pragma unroll
        for (int o = 0; o < NR; ++o) {
            float z = 0.0f;
#pragma unroll
            for (int a = 0; a < ALPHA; ++a) z = term<CO>(CO::at(tab, (O0 + o) * ALPHA + a), col[a], z);
#pragma unroll
            for (int p = 0; p < MM; ++p) Y[o][p] = term<CO>(CO::at(tab, p * ALPHA + b), z, Y[o][p]);
        }
    }
#pragma unroll
    for (int o = 0; o < NR; ++o) {
        const int64_t hr = hr0 + O0 + o;
        if (hr >= geo.H) break;
        Elem* dst = yk + (hr * geo.W + wc0) * geo.K;
#pragma unroll
        for (int p = 0; p < MM; ++p) {
            if (wc0 + p >= geo.W) break;
            dst[p * geo.K] = S::from_f32(Y[o][p]);
        }
    }
}

template <typename Elem, int MM, int ALPHA, class CO, int kG>
__global__ __launch_bounds__(kOutBlock) void output_transform_regs(OutputTable tab, const float* __restrict__ Mx,
                                                              Elem* __restrict__ y, Geometry geo, OutputMap mp) {
    const int64_t bid = blockIdx.x, G = gridDim.x;
    const int64_t xcd = bid % 8;
    const int64_t unit = xcd * (G / 8) + (xcd < G % 8 ? xcd : G % 8) + bid / 8;   // XCD-aware, as the input transform
    const int group = static_cast<int>(unit % kG);
    const int64_t gid = unit / kG * kOutBlock + threadIdx.x;
    if (gid >= mp.threads) return;
    const uint32_t tl = fast_div(static_cast<uint32_t>(gid), mp.per_tile);
    const int64_t k = static_cast<int64_t>(static_cast<uint32_t>(gid) - tl * mp.per_tile.d);
    const int64_t tile = mp.tile0 + tl;
    const uint32_t row = fast_div(static_cast<uint32_t>(tile), mp.tw);
    const uint32_t tx = static_cast<uint32_t>(tile) - row * mp.tw.d;
    const uint32_t n = fast_div(row, mp.th);
    const uint32_t ty = row - n * mp.th.d;
    const float* in = Mx + tile * geo.Kp + k;
    Elem* yk = y + static_cast<int64_t>(n) * geo.H * geo.W * geo.K + k;
    const int64_t plane = geo.T * geo.Kp, hr0 = static_cast<int64_t>(ty) * MM, wc0 = static_cast<int64_t>(tx) * MM;
    constexpr int kR = (MM + kG - 1) / kG;
    if (group == 0) output_regs_rows<Elem, MM, ALPHA, CO, 0, kR>(tab, in, plane, yk, hr0, wc0, geo);
    if constexpr (kR < MM)
        if (group != 0) output_regs_rows<Elem, MM, ALPHA, CO, kR, MM>(tab, in, plane, yk, hr0, wc0, geo);
}

}  // namespace wg
