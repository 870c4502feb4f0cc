// rlx_share.hpp -- how the waves of a batched launch share its items.
#pragma once
#include <cstdint>

namespace rlx {

// A plan with few items leaves most of the chip idle while one wave runs the
// longest of them (256 requests up to 65 536 values: 264 items, the longest 64
// iterations of a wave, 99 us of it), so waves share items: as many as keep
// those with work within SHARE_WAVES, twice what the chip holds, and each
// takes at least MIN_SHARE iterations, beside which its start-up is worth 3 to
// 10 steps.  The grid covers the plan's capacity and only bounds the share
// from above.  Measured on plans with room for 87 381 segments, unshared, by
// the whole grid, and so: 1000 requests of 1024 values 15, 84 and 10.6 us; of
// 8192 values, 10^8 values into their streams, 27, 206 and 26; 3660 requests
// up to 98 304 values 169, 109 and 97.  A server of such plans: 5.55e11,
// 5.32e11 and 5.99e11 doubles/s, at half load p99 0.76, 1.09 and 0.74 ms.
// With 12 288 waves 5.92e11 and 0.78 ms; with parts of 2 iterations 6.0e11 and
// 0.90 ms, the requests of 8192 values 31 us.
constexpr uint32_t SHARE_WAVES = 8192, MAX_SHARE = 64, MIN_SHARE = 4;

// Waves that share each of `n_items` items (at most the grid's waves).
constexpr uint32_t item_share(uint32_t n_items, uint32_t grid_waves) {
  const uint32_t waves = grid_waves < SHARE_WAVES ? grid_waves : SHARE_WAVES;
  const uint32_t share = waves / (n_items ? n_items : 1u);
  return share > MAX_SHARE ? MAX_SHARE : share ? share : 1u;
}

// Blocks of each of an item's segments that each of `share` waves takes, in
// whole iterations of 2^lgs blocks; `cost`: blocks of the item's longest
// segment.
constexpr uint32_t part_blocks(uint32_t cost, uint32_t lgs, uint32_t share) {
  const uint32_t its = (cost + (1u << lgs) - 1u) >> lgs;
  const uint32_t per = (its + share - 1u) / share;
  return (per > MIN_SHARE || share == 1 ? per : MIN_SHARE) << lgs;
}

}  // namespace rlx
