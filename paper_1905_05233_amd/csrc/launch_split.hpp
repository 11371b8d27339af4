// How layers too large for one launch are split (host arithmetic only).
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

}  // namespace wg
