// Which kernel aggregates the variables of a bf16 model with 2 x 2 patches and head dimensions that are multiples of 64
// (elementwise.hip): matrix instructions or the vector pipe.  Arithmetic only: the CPU test compiles it too and holds the choice
// against measured times.
#pragma once

namespace reslim {

// features, variables, patches of ONE sample: the two kernels round differently, and so a sample's tokens do not depend on its batch.
// The matrix kernel takes a step for every two variables and fills and drains its pipes around them: few variables do not pay for that, the
// less so the more features a work-group walks through (one variable at 256 features 6.6 us against 6.2 on the vector pipe, at 3072 28.9 and
// 14.7).  Up to 256 features two variables are enough (23 at 1024 patches: 14.8 and 25.8), below 1024 seven (five at 512 features and
// 1024 patches 10.9 and 10.1, eight 11.9 and 12.3).  From 1024 features on the vector kernel takes 16 patches an item, which keeps
// up until the chip is full (1024 features, 23 variables: 4096 patches 50 and 46, 16,384 68 and 71, 65,536 209 and 234; 3072
// features, 16 variables: 96 and 91 at 4096, 139 and 210 at 16,384); where the features are no multiple of 1024 those items leave threads idle.
inline bool embed_on_matrix_pipe(int features, int variables, long long patches) {
  if (features <= 256) return variables >= 2;
  if (features < 1024) return variables >= 7;
  if (features < 2048 && features % 1024 != 0) return variables >= 8;
  if (patches < 16000) return variables >= 32;
  return variables >= (features < 2048 || patches >= 65000 ? 8 : 16);
}

}  // namespace reslim
