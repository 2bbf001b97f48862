// GELU of the bf16 path and the conversion of its results, shared by the kernels that apply it (gemm.hip, panel.hip).
#pragma once

#include "common.h"

namespace reslim {

// GELU for bf16 outputs without the reciprocal and the branches of the library erf: with u = min(|x|, 5), Phi(-u) = 2^P(u) where P
// is a degree-6 fit of log2 of the normal tail on [0, 5] (interpolated at Chebyshev nodes), and gelu(x) = max(x, 0) - u Phi(-u).
// Relative error <= 1.5e-5 of gelu(x) for |x| <= 5, against 2^-9 for the bf16 rounding that follows; absolute error <= 2e-6
// for every x (1.91e-6 at |x| = 1), and 1.43e-6 below -5, where the result stays what it is at -5.  A degree-5 fit of the absolute error
// saves one of the 10 vector operations, and halves that error, but is off by 2^-9 of the result at -4.5 and by 1.2 % at -5.
// Both bounds are v_med3_f32: fminf and fmaxf of a matrix result cost a second operation each that quiets signalling NaNs.
__device__ __forceinline__ float gelu_erf_fast(float x) {
  const float u = __builtin_amdgcn_fmed3f(fabsf(x), 0.0f, 5.0f);
  float p = fmaf(2.975744064e-05f, u, -7.135751075e-04f);
  p = fmaf(p, u, 7.775241509e-03f);
  p = fmaf(p, u, -5.269032717e-02f);
  p = fmaf(p, u, -4.595123231e-01f);
  p = fmaf(p, u, -1.150926590e+00f);
  p = fmaf(p, u, -1.000011683e+00f);
  return fmaf(-u, __builtin_amdgcn_exp2f(p), __builtin_amdgcn_fmed3f(x, 0.0f, 3.402823466e+38f));
}

// two floats -> two bf16 in one register (one hardware conversion)
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

}  // namespace reslim
