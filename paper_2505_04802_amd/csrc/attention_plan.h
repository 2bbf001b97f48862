// Which kernel tile attention at head dimension 64 takes (attention.hip): keys split over the waves, 32 queries a wave, or 64.  Arithmetic only: the
// CPU test compiles it too and holds the choice against measured times.
#pragma once

#include <cstdint>

namespace reslim {

// Work-groups that one launch may have: a dimension of a grid takes fewer than 2^32 threads.  More slots than that are many short tiles, or sequences of which
// one is long: the forward takes its persistent kernel, the gradient several launches.
constexpr int64_t most_work_groups(int threads) { return 0xffffffffLL / threads; }

// units: of 128 queries, over the whole launch; cus: compute units; tokens: of the longest tile.
// The split kernel has four work-groups to a unit, two at a time on a compute unit.  Up to half as many units as compute units
// they all run at once, and it is 1.2 to 2.6 times as fast from 512 tokens on (512 tokens, 128 units: 12.0 us without the split,
// 9.2 with; 2300 tokens, 72 units: 41 and 22; shorter tiles leave a wave two blocks).  With more, the second round is partly empty
// while the other kernel still needs the time of one unit: 768 tokens, 192 units: 16.4 and 16.1; 1440, 192: 27.8 and 26.8; 512,
// 192: 12.2 and 13.1.  From there to one unit a compute unit only long tiles gain: 2300 tokens, 234 units: 41.5 and 40.6; 1806, 240: 34.2
// and 34.5; 1024, 224: 20.6 and 21.9.  Past that every wave of the chip has work without the split, and it loses a quarter or more.
inline bool attn_split_keys(int units, int cus, int tokens) {
  if (tokens < 512 || units > cus) return false;
  if (units <= cus / 2) return true;
  return tokens >= (units <= cus * 3 / 4 ? 768 : 2048);
}

// Waves in a work-group of the kernel with two query groups a wave, 0: the kernel with one.
// Both give the same bits.  u128, u256: tokens of all tiles, samples and heads in blocks of 128 and of 256 queries; cus: compute units; tokens: of the longest tile.
// Where every SIMD has work for two waves and more, two groups a wave are 1.05 to 1.2 times as fast (blocks of 128 queries per compute unit in
// brackets; one group, two): 1290 tokens, 512 sets of keys (22) 276 and 251 us; 660, 1024 (24) 189 and 159; 2000, 64 (4) 89 and 73; 400, 256 (4) 26.8 and
// 23.5.  One group a wave keeps three blocks on a compute unit, two groups four and half as many waves to give them.  Up to three blocks all
// run at once either way and the smaller waves spread better: 2000 tokens, 16 sets (1) 37.1 and 39.5; 1000, 64 (2) 26.7 and 27.8; 1290, 64 (2.75) 40.3 and
// 45.1; 660, 128 (3) 25.6 and 29.0.  From four to four and a half the second round of two groups is nearly empty: 1290, 96 (4.1) 63.8 and 66.9; 660,
// 192 (4.5) 39.8 and 41.6; 1290, 128 (5.5) 76.2 and 71.2.
// Four waves share a block of keys, which takes half the loads, but those without queries at a tile's end keep their place to the end of it: four only
// where they are at most a tenth more than in blocks of 128 (520 tokens, 512 sets, a fifth more: 64 us with one group, 71 with two; 300, 1024, a
// third more: 49 and 65; 1290, 256, a tenth more: 143 and 132).  Two waves leave fewer idle and are twice as many work-groups to start: for
// launches of 32 blocks a compute unit and more, where that leaves a twentieth fewer waves (tiles of 1274 to 1643 tokens, 203 blocks: 2.77 ms
// with four, 2.71 with two; 520 tokens, 40 blocks 249 us with one group, 226 with two waves of two; 1290 tokens, 11 blocks 132 with four, 139).
// Up to 40 tokens the second group has no or few queries and a tile is over with the first two blocks of keys (16,384 sets: 33 tokens 83.7 us with one group, 88.8 with
// two, 40 tokens 102.7 and 102.1, 48 118.9 and 109.9; 8192 sets of 48 46.1 and 48.4, of 64 56.3 and 53.3).
inline int attn_pair_waves(int64_t u128, int64_t u256, int cus, int tokens) {
  if (tokens <= 40) return 0;
  if (u128 <= 3LL * cus || (u128 > 4LL * cus && 2 * u128 <= 9LL * cus)) return 0;
  if (u128 >= 32LL * cus && 20 * u128 <= 19 * 2 * u256) return 2;
  return 10 * 2 * u256 <= 11 * u128 ? 4 : 0;
}

}  // namespace reslim
