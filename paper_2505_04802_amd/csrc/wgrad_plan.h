// Which tile and how many slices of the tokens the weight gradients of a launch get (wgrad.hip).  Arithmetic only: the CPU
// test compiles it too, to know which kernel a shape takes.
#pragma once

#include <initializer_list>
#include <stdint.h>

namespace reslim {

// Parameter gradients of linear layers over the same M tokens, up to kWgradMax of them at once:
// dW[N, K] = dY[M, N]^T X[M, K] and db[N] = column sums of dY, both fp32; ws >= wgrad_ws_bytes
constexpr int kWgradMax = 4;
struct WgradOp {
  const void *dy, *x;
  float *dw, *db;
  int N, K;
};

enum WgradKind { kWgrad128x256, kWgrad256 };
struct WgradPlan { WgradKind kind; int tiles, splits, m_per_split; };
inline int wgrad_tiles_n(WgradKind kind, int N) { return kind == kWgrad256 ? (N + 255) / 256 : (N + 127) / 128; }
inline WgradPlan wgrad_split(WgradKind kind, const WgradOp *op, int n_op, int M, int splits) {
  WgradPlan p;
  p.kind = kind;
  p.tiles = 0;
  for (int i = 0; i < n_op; ++i) p.tiles += wgrad_tiles_n(kind, op[i].N) * ((op[i].K + 255) / 256);
  p.m_per_split = ((M + splits - 1) / splits + 63) / 64 * 64;
  p.splits = (M + p.m_per_split - 1) / p.m_per_split;
  return p;
}
inline int64_t wgrad_slice(const WgradOp *op, int n_op) {      // floats of one slice of partial sums
  int64_t n = 0;
  for (int i = 0; i < n_op; ++i) n += (static_cast<int64_t>(op[i].K) + 1) * op[i].N;
  return n;
}
// Tile and slices by estimated time (us), fitted to measured launches of one to four products, 130 to 97,760 tokens and
// 96 to 16,384 features: a slab of 64 tokens takes a work-group 0.95 us at 128 x 256 (bound by the feed of LDS) and 1.65 us at
// 256 x 256 (matrix cores, on large launches the power limit), a round of work-groups (one per CU) 2 us to fill its pipeline,
// and a slice of partial sums 0.31 us per MB to write and add up, after 4 us for the second launch.
inline WgradPlan wgrad_plan(const WgradOp *op, int n_op, int M, int cus) {
  const double mb = 4e-6 * static_cast<double>(wgrad_slice(op, n_op));
  WgradPlan best = {};
  double best_t = 0;
  for (WgradKind kind : {kWgrad256, kWgrad128x256}) {
    const int tiles = wgrad_split(kind, op, n_op, M, 1).tiles;
    const int cap = 4 * cus / tiles > 1 ? 4 * cus / tiles : 1;      // up to four rounds, if that ends in a full one
    for (int s = 1; s <= cap; ++s) {
      const WgradPlan p = wgrad_split(kind, op, n_op, M, s);
      const int rounds = static_cast<int>((static_cast<int64_t>(tiles) * p.splits + cus - 1) / cus);
      const double t = rounds * (2.0 + p.m_per_split / 64 * (kind == kWgrad256 ? 1.65 : 0.95)) + (p.splits > 1 ? 4.0 + 0.31 * mb * p.splits : 0.0);
      if (best.tiles == 0 || t < best_t) {
        best = p;
        best_t = t;
      }
    }
  }
  return best;
}

}  // namespace reslim
