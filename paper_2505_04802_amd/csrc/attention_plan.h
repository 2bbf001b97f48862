// When tile attention at head dimension 64 splits the keys over the waves of a work-group (attention.hip).  Arithmetic only: the
// CPU test compiles it too and holds the choice against measured times.
#pragma once

namespace reslim {

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

}  // namespace reslim
