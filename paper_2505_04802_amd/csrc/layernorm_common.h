// The arithmetic of LayerNorm, shared by the kernels that apply it to whole rows (elementwise.hip) and to rows that lie
// across the waves of a work-group (panel.hip).  At the widths that both take they have to give the same bits, so the order is fixed here: four consecutive
// columns first (below), then 32 columns (lanes 2, 4, then 1 apart where a lane holds four columns), then 64, 128 and
// 256, then the 256-column pieces of the row from the first on.  Contractions are written out: left to the compiler they would depend on the
// code around them.
#pragma once

#include "common.h"

namespace reslim {

__device__ __forceinline__ float ln_sum4(float a, float b, float c, float d) { return (a + b) + (c + d); }
__device__ __forceinline__ float ln_square4(float a, float b, float c, float d) { return fmaf(a, a, b * b) + fmaf(c, c, d * d); }
__device__ __forceinline__ float ln_rstd(float sq, float D) { return rsqrtf(sq / D + 1e-5f); }
__device__ __forceinline__ float ln_apply(float v, float mean, float rstd, float gain, float bias) { return fmaf((v - mean) * rstd, gain, bias); }

// sum over the lanes of a wave, each holding four consecutive columns
__device__ __forceinline__ float ln_lane_sum(float s) {
  s += __shfl_xor(s, 2);
  s += __shfl_xor(s, 4);
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 8);
  s += __shfl_xor(s, 16);
  s += __shfl_xor(s, 32);
  return s;
}

}  // namespace reslim
