// How layers too large for one launch are split, and which form of the 1D and the
// float64 convolution a layer takes (host arithmetic only).
//
// HIP takes launches of fewer than 2^32 work-items along x (gridDim.x *
// blockDim.x), whatever the ids that the kernel itself computes.
#pragma once

#include <algorithm>
#include <cstdint>

namespace wg {

constexpr int64_t kMaxWorkItems = 0xffffffff;

// Output transform in registers: workgroups of kOutBlock (tile, channel) pairs,
// `groups` of them (row groups, kOutGroups at most) for the same pairs.
constexpr int kOutBlock = 256;
constexpr int kOutGroups = 2;
// Most pairs of a launch: ids below 2^31, and the row groups' workgroups within
// kMaxWorkItems.
constexpr int64_t output_max_pairs(int groups) {
    return std::min<int64_t>(0x7fffffff, kMaxWorkItems / groups) / kOutBlock * kOutBlock;
}
// Whole tiles of one launch for K output channels (K at most output_max_pairs), and
// its workgroups for `pairs` pairs.
constexpr int64_t output_tiles_per_launch(int64_t K, int groups) { return output_max_pairs(groups) / K; }
constexpr int64_t output_blocks(int64_t pairs, int groups) { return (pairs + kOutBlock - 1) / kOutBlock * groups; }

// Input transform in registers: 32-bit offsets into the pixels that a launch
// reads, at most kInMaxBytes of them (below the out-of-range offsets that its
// kernel uses), thread ids below 2^31, and the row groups' workgroups within
// kMaxWorkItems.
constexpr int kInBlock = 256;
constexpr int64_t kInMaxBytes = int64_t(1) << 30;
constexpr int64_t input_max_threads(int groups) {
    return std::min<int64_t>(0x7fffffff, kMaxWorkItems / groups / kInBlock * kInBlock);
}
constexpr int64_t input_blocks(int64_t threads, int groups) { return (threads + kInBlock - 1) / kInBlock * groups; }
// What one launch covers: `images` whole images, or, where one image is too
// large, `rows` tile rows of one.  rows = 0: not even one tile row fits.
struct InputSplit {
    int64_t images, rows;
};
// row_bytes: of a row of pixels; tile_row_threads: threads of a row of tiles;
// groups: the row groups of layers of any size.
constexpr InputSplit input_split(int64_t H, int64_t row_bytes, int64_t tile_rows, int64_t tile_row_threads, int m,
                                 int groups) {
    const int64_t img_bytes = H * row_bytes, img_threads = tile_rows * tile_row_threads, most = input_max_threads(groups);
    if (img_bytes <= kInMaxBytes && img_threads <= most)
        return {std::min<int64_t>(kInMaxBytes / img_bytes, most / img_threads), tile_rows};
    // r tile rows read at most r m + 2 rows of pixels
    const int64_t rows = std::min<int64_t>((kInMaxBytes / row_bytes - 2) / m, most / tile_row_threads);
    return {1, std::max<int64_t>(0, std::min(rows, tile_rows))};
}
// The rows of pixels that tile rows r0 .. r0 + rows - 1 read: [first, end).
struct InputBand {
    int64_t first, end;
};
constexpr InputBand input_band(int64_t H, int64_t r0, int64_t rows, int m) {
    return {std::max<int64_t>(0, r0 * m - 1), std::min<int64_t>(H, (r0 + rows) * m + 1)};
}

// 1D form: workgroups of the one kernel (conv1d.hip), k1dWaves waves that own 16 kw
// output channels x 32 (k1dWaves / kw) tiles and walk the channels in chunks.
constexpr int k1dWaves = 8;
constexpr int k1dChunk = 64;             // bytes of a channel row per step
constexpr int conv1d_waves_k(int64_t K) { return K > 64 ? 8 : 4; }
constexpr int64_t conv1d_chunks(int64_t Cp, int64_t es) { return (Cp * es + k1dChunk - 1) / k1dChunk; }
constexpr int64_t conv1d_k_blocks(int64_t K) { return (K + 16 * conv1d_waves_k(K) - 1) / (16 * conv1d_waves_k(K)); }
constexpr int64_t conv1d_blocks(int64_t T, int64_t K) {
    const int64_t n_tiles = 32 * (k1dWaves / conv1d_waves_k(K));
    return (T + n_tiles - 1) / n_tiles * conv1d_k_blocks(K);
}

// Where the one kernel is the faster form.
//
// It walks a row's chunks one after another, so a layer with long rows and few
// blocks is faster through the separate kernels, which spread the points over the
// chip: 1x100, 512 -> 512 in bf16 (4 blocks, 16 chunks) 40 against 21 us, 8x512,
// 512 -> 512 (128 blocks) 42 against 40 us; one of few chunks is not (3x6542, 16 ->
// 16 6 against 16 us).  Every block of output channels transforms the input anew
// and holds its operands in small tiles, so layers that are wide and deep go
// through the separate kernels too: their two times are estimated (in ns) from the
// rounds of blocks that the one kernel takes, and from V, M and the products of
// the separate ones.  Fitted to 1364 layers (N 1 - 64, L 16 - 8000, C 8 - 512, K 8 -
// 1024, alpha' 4, 6, 7 and 10, fp32 and 16 bits), of which the worst choices with up
// to 512 output channels lose 9 % (8000 positions, 512 -> 512, alpha' = 4 in fp32)
// and 10 % (5x8000, 301 -> 77, alpha' = 7 in fp32), beyond 17 %.  One kernel and
// separate: alpha' = 7 in fp16, 16x4096, 128 -> 128 26 and 87 us; alpha' = 10 in fp32,
// 5x8000, 128 -> 512 173 and 146 us, 16x4096, 512 -> 512 901 and 633; in fp16 64x300,
// 512 -> 1024 258 and 140 us.
constexpr int64_t k1dFewPoints = 20;    // chunks x alpha' that one block may walk anyway
constexpr int64_t k1dBlocksPerChunk = 14;
constexpr bool conv1d_one_kernel_pays(int64_t T, int64_t Cp, int64_t K, int64_t Kp, int alpha, int64_t es) {
    const int64_t ch = conv1d_chunks(Cp, es), blocks = conv1d_blocks(T, K);
    if (ch * alpha <= k1dFewPoints) return true;
    if (blocks < k1dBlocksPerChunk * ch) return false;
    const double a = alpha, n = static_cast<double>(ch), cols = static_cast<double>((K + 127) / 128);
    const double pts = 1e-3 * a * static_cast<double>(T), cp = static_cast<double>(Cp), kp = static_cast<double>(Kp);
    // blocks at once: two per CU where the registers allow it (launch bounds of the kernel)
    const int64_t slots = es == 2 && alpha <= 7 ? 512 : 256;
    const double rounds = static_cast<double>((blocks + slots - 1) / slots);
    if (es == 2)
        return 5500 + rounds * (420 + 630 * n + a * (310 * n + 490)) <= 20400 + pts * (2.0 * cp + 1.7 * kp + 9.8 * n * cols);
    return 6900 + rounds * (n * (540 * a - 640) + 380 * a) <=
           21400 + pts * (1.8 * cp + 1.7 * kp + (ch <= 8 ? 25.5 : 32.0) * n * cols);
}

// Float64 direct convolution: one thread per output, or the matrix cores with
// 32 x 32, 64 x 64 or 128 x 32 (pixels x output channels) outputs per workgroup.
enum F64Form { kF64PerOutput, kF64Block32, kF64Block64, kF64Block128x32 };
// taps: 9 or 3; es: bytes of a value.  The matrix cores where a block's columns
// and chunk are mostly filled and 32-bit offsets reach both inputs; small layers
// in 32 x 32 outputs, for more workgroups.
constexpr F64Form f64_form(int64_t pixels, int64_t C, int64_t K, int taps, int64_t es, int cus) {
    const int64_t R = taps * C;
    if (!(K > 8 && R > 16 && R < (int64_t(1) << 30) && pixels * C * es < 0xfffffff0LL && K * R * es < 0xfffffff0LL &&
          pixels / 32 < 0x7fffffff && K / 32 < 0xffff))
        return kF64PerOutput;
    const int64_t bn = K > 32 ? 64 : 32, bm = 4096 / bn;
    if (((pixels + bm - 1) / bm) * ((K + bn - 1) / bn) < cus / 2) return kF64Block32;
    return bn == 64 ? kF64Block64 : kF64Block128x32;
}

}  // namespace wg
