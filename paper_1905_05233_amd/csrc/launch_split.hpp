// How layers too large for one launch are split, and which form of the float64
// convolution a layer takes (host arithmetic only).
//
// HIP takes launches of fewer than 2^32 work-items along x (gridDim.x *
// blockDim.x), whatever the ids that the kernel itself computes.
#pragma once

#include <algorithm>
#include <cstdint>

namespace wg {

constexpr int64_t kMaxWorkItems = 0xffffffff;

// Output transform in registers: workgroups of kOutBlock (tile, channel) pairs,
// kOutGroups of them (row groups) for the same pairs.
constexpr int kOutBlock = 256;
constexpr int kOutGroups = 2;
// Most pairs of a launch: ids below 2^31, and the row groups' workgroups within
// kMaxWorkItems.
constexpr int64_t kOutMaxPairs =
    std::min<int64_t>(0x7fffffff, kMaxWorkItems / kOutGroups) / kOutBlock * kOutBlock;
// Whole tiles of one launch for K output channels (K at most kOutMaxPairs), and
// its workgroups for `pairs` pairs.
constexpr int64_t output_tiles_per_launch(int64_t K) { return kOutMaxPairs / K; }
constexpr int64_t output_blocks(int64_t pairs) { return (pairs + kOutBlock - 1) / kOutBlock * kOutGroups; }

// Input transform in registers: 32-bit offsets into the pixels that a launch
// reads, at most kInMaxBytes of them (below the out-of-range offsets that its
// kernel uses), and thread ids below 2^31.
constexpr int kInBlock = 256;
constexpr int64_t kInMaxBytes = int64_t(1) << 30;
// What one launch covers: `images` whole images, or, where one image is too
// large, `rows` tile rows of one.  rows = 0: not even one tile row fits.
struct InputSplit {
    int64_t images, rows;
};
// row_bytes: of a row of pixels; tile_row_threads: threads of a row of tiles.
constexpr InputSplit input_split(int64_t H, int64_t row_bytes, int64_t tile_rows, int64_t tile_row_threads, int m) {
    const int64_t img_bytes = H * row_bytes, img_threads = tile_rows * tile_row_threads;
    if (img_bytes <= kInMaxBytes && img_threads <= 0x7fffffff)
        return {std::min<int64_t>(kInMaxBytes / img_bytes, 0x7fffffff / img_threads), tile_rows};
    // r tile rows read at most r m + 2 rows of pixels
    const int64_t rows = std::min<int64_t>((kInMaxBytes / row_bytes - 2) / m, 0x7fffffff / tile_row_threads);
    return {1, std::max<int64_t>(0, std::min(rows, tile_rows))};
}
// The rows of pixels that tile rows r0 .. r0 + rows - 1 read: [first, end).
struct InputBand {
    int64_t first, end;
};
constexpr InputBand input_band(int64_t H, int64_t r0, int64_t rows, int m) {
    return {std::max<int64_t>(0, r0 * m - 1), std::min<int64_t>(H, (r0 + rows) * m + 1)};
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
