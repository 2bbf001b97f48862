// When the panel kernel (panel.hip) takes a block, and how many rows a work-group of it.  Arithmetic only: the CPU test compiles it too.
#pragma once

namespace reslim {

// Widths that the panel kernel is made for, 32 columns times eight waves times one or two.
inline bool panel_width(int D) { return D == 256 || D == 512; }

// Rows from which one launch beats the separate ones (a block's time, the same forward captured with either form).  A panel cannot take
// less than the time in which the weights stream through a compute unit, R / D of them in the hidden layer.  At D = 256 that never loses: 32
// rows 44 us against 29 at R = 4 D, 68 against 57 at 16 D.  At D = 512 it grows by 9 us a D of the hidden layer, the separate launches
// by 4, and by 4 a thousand rows: R = 2 D 62 us against 59 at 1024 rows; 3 D 69 against 70 at 1024 and 72 against 70 at 1536; 4 D 71 against
// 78 at 1024, 76 and 78 at 2048, 80 and 78 at 2304; 8 D 88 and 115 at 1024, 113 and 118 at 4096, 133 and 123 at 6144.
inline int panel_rows_from(int D, int R) {
  if (D == 256) return 1;
  const int line = static_cast<int>(265LL * R / 128 - 2120);
  return line > 1024 ? line : 1024;
}

// Row blocks of 32 a panel has, one to three.  A panel's registers fill a compute unit, so what counts is rounds of panels times the
// time of one, part of it fixed (the weights stream through whatever the rows): 1.4 + rb.  Many rounds of one, two and three row blocks take 27, 39
// and 55 us each at D = 256, of one and two 80 and 113 at D = 512; a single round, all panels in step, 31, 41 and 54, and 86 and 113.
// 19,552 rows of 256 features take 75 us in panels of 32 (three rounds), 65 in panels of 64 (two) and 49 in panels of 96 (one).
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
