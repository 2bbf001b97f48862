// When the panel kernel (panel.hip) takes a block, and how many rows a work-group of it.  Arithmetic only: the CPU test compiles it too.
#pragma once

namespace reslim {

// Widths that the panel kernel is made for, 32 columns times eight waves times one or two.
inline bool panel_width(int D) { return D == 256 || D == 512; }

// Rows from which one launch beats the separate ones.  A panel cannot take less than the time in which the weights stream through a
// compute unit: 13 us at D = 256, where a block of 64 rows takes 27 us against 41, and 54 us at D = 512, where one of 512
// rows takes 67 us against 62, of 1024 rows 66 against 67 and of 2304 rows 70 against 75.
inline int panel_rows_from(int D) { return D == 256 ? 1 : 1024; }

// Row blocks of 32 a panel has, one to three.  A compute unit works on one panel at a time, so what counts is rounds of panels
// times the time of one, part of it fixed (the weights stream through whatever the rows).  At D = 256, 256 panels of one, two and three
// row blocks take 26, 37 and 49 us, so 1.4 + rb; 19,552 rows take 65 us in panels of 32, 58 in panels of 64 (two rounds either
// way but for a few) and 43 in panels of 96 (one round).
inline int panel_row_blocks(int M, int num_cus, int most) {
  int best = 1;
  double t_best = 0;
  for (int rb = 1; rb <= most; ++rb) {
    const long long panels = (static_cast<long long>(M) + 32 * rb - 1) / (32 * rb), rounds = (panels + num_cus - 1) / num_cus;
    const double t = static_cast<double>(rounds) * (1.4 + rb);
    if (rb == 1 || t <= t_best) {
      best = rb;
      t_best = t;
    }
  }
  return best;
}

}  // namespace reslim
