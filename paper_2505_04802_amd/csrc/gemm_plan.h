// Which bf16 kernel a product C[M, N] = A[M, K] W[N, K]^T gets (gemm.hip).  Arithmetic only: the CPU test compiles it too
// and holds the choice against measured times.
#pragma once

#include <algorithm>
#include <cmath>

namespace reslim {

enum GemmKernel { kGemm128 = 2, kGemm256x256 = 3, kGemm128x256 = 4 };      // one tile per work-group; persistent
// What an epilogue costs: bf16 output; with GELU; two bf16 outputs; fp32 output; fp32 output that reads as much again
enum GemmEpi { kEpiAct, kEpiGelu, kEpiTwo, kEpiF32, kEpiStream };

// The smallest of three estimates, in microseconds beside what every launch costs.  A round of the persistent kernels is
// one tile per CU: its 64-deep slabs and an epilogue, cheaper when part of the chip is idle.  The small tiles lie up to
// three on a CU and share it; past that nothing ties their work-groups together, so there is no last round.  Half of the CUs
// with a second (third) tile already cost most of what all of them do, hence the mean of w and its ceiling.
// Fitted to 4088 products (M 120 .. 160,000, N 64 .. 16,384, K 64 .. 8192, every epilogue) timed with all three kernels on
// MI355X.  On 6608 others the pick is within 0.7 % of the best of the three on average and more than 10 % behind in 1.5 % of
// them; with constants fitted to 52 products of mostly large M it was 2.2 %, and 9 %: short products went to the persistent
// kernels, whose start costs more than their slabs save there (392 x 2048 x 512 with GELU 0.012 ms with small tiles, 0.015 with
// 128 x 256).  In words: 256 x 256 tiles where there are at least about two rounds of them; 128 x 256 where their rounds come out emptier
// (42,560 x 512 x 2048: 0.124 -> 0.106 ms) or K is deep and there is less than one (5000 x 1024 x 4096: 0.072 -> 0.047); 128 x 128
// for shallow products with heavy epilogues, and for less than a round of shallow ones.
// The persistent kernels have to promise something: 2 us, and where they fill the chip 15 % or 4 us more, whichever is less.  On some chips a
// persistent launch that starts on all CUs at once lowers the clock by 7 % for the launches around it, short as it may be; one
// product of 16,200 x 512 x 512 in a forward of 0.70 ms that has no other costs 0.05 ms there, and saves 2 us.  Long products run at
// the power limit anyway.
inline GemmKernel gemm_choose(int M, int N, int K, GemmEpi epi, int num_cus) {
  constexpr double small_epi[] = {3.3, 3.32, 5.4, 5.99, 6.17}, pp2_epi[] = {4.81, 9.5, 13.97, 6.33, 11.12}, pp1_epi[] = {3.72, 5.25, 8.53, 3.41, 6.76};
  const double nk = K / 64, cus = num_cus;
  auto tiles = [&](int bm, int bn) { return static_cast<double>((M + bm - 1) / bm) * ((N + bn - 1) / bn) / cus; };      // per CU
  const double w2 = tiles(256, 256), w1 = tiles(128, 256), ws = tiles(128, 128);
  const double f2 = std::min(1.0, w2), f1 = std::min(1.0, w1);                             // share of the chip at work
  const double fs = std::min(1.0, std::max(0.0, (0.62 * std::ceil(ws) + 0.38 * ws - 1.0) / 2.0));
  auto promise = [](double c, double w) { return c + 2.0 + (w >= 0.85 ? std::min(4.0, 0.15 * c) : 0.0); };
  const double c2 = promise(2.46 + std::ceil(w2) * (nk * (1.08 + 0.10 * f2) + pp2_epi[epi] * (0.36 + 0.64 * f2)), w2);
  const double c1 = promise(0.34 + std::ceil(w1) * (nk * (0.43 + 0.30 * f1) + pp1_epi[epi]), w1);
  const double cs = std::max(1.0, ws / 3.0) * (nk * (0.73 + 1.07 * fs) + small_epi[epi] * (0.12 + 0.88 * fs));
  return cs <= c1 && cs <= c2 ? kGemm128 : c1 < c2 ? kGemm128x256 : kGemm256x256;
}

// fp32 path: whether a product M x N x K normalises its rows itself (gemm_f32_kernel with LN) instead of after a launch of its own.
// Every column tile of the outputs repeats the LayerNorm, which is free while a compute unit has no more than three tiles of 32 x 32: it saves
// 1 to 2 us then (512 x 384 x 128: 1.6; 2048 x 384 x 128, 768 tiles: 0.3).  With more it costs up to 4 (4096 x 384 x 128, 1536 tiles: 2.8; 1536 x
// 768 x 96, 1152 tiles: 3.8), but for products with no more columns than features, which repeat it too seldom to notice (8192 x
// 64 x 64, 512 tiles: saves 3.2; 12,288 x 160 x 160, 1920 tiles: 2.4).
inline bool gemm_f32_normalises(int M, int N, int K, int num_cus) {
  const long long tiles = static_cast<long long>((M + 31LL) / 32) * ((N + 31LL) / 32);
  return tiles <= 3LL * num_cus || ((N <= K || N <= 32) && tiles < 8LL * num_cus);
}

}  // namespace reslim
