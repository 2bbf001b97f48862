// GELU of the bf16 path and the conversion of its results, shared by the kernels that apply it (gemm.hip, panel.hip).
#pragma once

#include "common.h"

namespace reslim {

// GELU for bf16 outputs without the reciprocal and the branches of the library erf: with u = |x|, Phi(-u) = 2^P(u) where P
// is a degree-5 fit of log2 of the normal tail, and gelu(x) = max(x, 0) - u Phi(-u).  Absolute error <= 1e-6 for every x (0.97e-6 at
// most, near |x| = 0.4; 2e-8 beyond 5), 4.3e-6 (inputs of standard deviation 0.3) to 2.0e-7 (of 4) of the result in the root mean square, against
// 2^-9 for the bf16 rounding that follows.  The fit weighs absolute errors: a degree-6 one of constant relative error
// (1.3e-5 up to 5) was up to 1.9e-6 off, 4.4e-6 to 3.1e-7 in the mean, and cost one vector operation more; this one is up to
// 1.2 % off where the result is below 1e-6.  P falls without bound, so the limit on u only keeps
// infinities out of the last product.  Both bounds are v_med3_f32: fminf and fmaxf of a matrix result cost a second operation each
// that quiets signalling NaNs.  9 vector operations, one of them an exponential of twice the time.
__device__ __forceinline__ float gelu_erf_fast(float x) {
  const float u = __builtin_amdgcn_fmed3f(fabsf(x), 0.0f, 64.0f);
  float p = fmaf(-4.180783580522984e-04f, u, 6.723981350660324e-03f);
  p = fmaf(p, u, -5.0993356853723526e-02f);
  p = fmaf(p, u, -4.608226716518402e-01f);
  p = fmaf(p, u, -1.1504477262496948e+00f);
  p = fmaf(p, u, -1.0000799894332886e+00f);
  return fmaf(-u, __builtin_amdgcn_exp2f(p), __builtin_amdgcn_fmed3f(x, 0.0f, 3.402823466e+38f));
}

// two floats -> two bf16 in one register (one hardware conversion)
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}

}  // namespace reslim
