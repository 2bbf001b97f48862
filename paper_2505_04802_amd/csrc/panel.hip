// The part of a transformer block that works on each token by itself, as ONE launch (ORBIT-2 Sec. 3 / 4.1):
//   x_mid = x + proj(attention output);  x' = x_mid + fc2(gelu(fc1(ln2(x_mid))));
//   and, where another block follows, its qkv = ln1'(x') W^T + b.
// bf16 path, for models whose rows fit a compute unit: a work-group takes a PANEL of 32 RB whole rows through all of it.
//
// Why it is one kernel.  At D = 256 the products and LayerNorms of a block are launches of 8 to 24 us each: outputs of one
// or two column tiles leave the products at 250-550 TFLOP/s, and the hidden layer, qkv and the stream go through memory between
// them.  In one launch the rows stay in registers and LDS and only the weights stream in, 1.6 MB a panel at D = 256 and 6.3 MB at 512,
// which a compute unit takes from L2 at 110 bytes a nanosecond.  What it measured (MI355X, with the next qkv): 19,552 rows of 256
// features 91 us in seven launches, 47 here (204 panels of 96 rows: 653 TFLOP/s); 42,560 rows of 512 384 us, 325 here (823).
// What bounds it: the matrix pipe is busy 42 % of the time at D = 256 and shares the SIMD with the vector work of GELU, LayerNorm and
// addresses (two waves' matrix and vector instructions take the sum of the one and half the other at best); panels of 32 rows
// wait for the weights.
//
// Weights are packed once, when the context is made, in the order in which the waves consume them: a fragment (32 output
// columns x 16 k, the A operand of one v_mfma_f32_32x32x16_bf16) is one contiguous KiB that goes from L2 straight into
// registers, PF fragments ahead of their use.  Every wave owns other columns, so no weight is fetched twice and no barrier
// is needed for them.  The activations are the operand that all waves share; they lie in LDS as rows whose 16-byte chunk c
// is at position c ^ (row & 15): conflict-free for the 16-byte fragment reads of 16 rows.
//
// The hidden layer is taken in chunks of CH columns through two LDS buffers.  GELU of chunk c is placed between the matrix instructions of
// FC2 of chunk c - 1 and FC1 of chunk c + 1 (51 us without, 46 with), and the order in which LDS reads, matrix and vector
// instructions of a step are issued is pinned (43).
//
// Every result is the same bits as that of the separate kernels: a product sums k upwards from zero in one accumulator, then comes the
// bias, then the skip connection; GELU and LayerNorm are shared (gelu.h, layernorm_common.h).  So it does not matter to a
// result which of the two forms a call takes, by its rows, its batch or its alignment.  Sums that start from the skip connection and
// the bias need no second set of registers, but their rounding grows with the stream; they would be 2 % faster (46.2 and 47.1 us
// side by side for 19,552 rows of 256 features, 322 and 325 for 42,560 of 512).
#include <type_traits>
#include <utility>

#include "attention_common.h"
#include "gelu.h"
#include "layernorm_common.h"
#include "panel_plan.h"

namespace reslim {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct Nothing {
  template <class I>
  __device__ __forceinline__ void operator()(I) const {}
};

// f(0) .. f(N - 1) with compile-time numbers: `#pragma unroll` gives up on bodies of this size
template <class F, int... I>
__device__ __forceinline__ void each_of(F &&f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each(F &&f) {
  each_of(f, std::make_integer_sequence<int, N>{});
}

struct PanelArgs {
  const bf16_t *a;         // [M, D] attention output
  const float *res;        // stream before the block: row m, or the row that res_map names (see ResRowMap)
  const int32_t *res_map;
  int res_out;
  int64_t res_in;
  float *x;                // [M, D] stream after the block (may be res)
  bf16_t *qkv;             // [M, 3 D], null: no next block
  const bf16_t *w;         // packed matrices that this launch reads
  unsigned w_bytes;
  int w_proj, w_fc1, w_fc2, w_qkv;      // byte offsets in them
  const float *b_proj, *b_fc1, *b_fc2, *b_qkv, *ln2_g, *ln2_b, *ln1_g, *ln1_b;
  int M, R;
  float qscale;            // factor of the first D columns of qkv
};

// NW waves, NB column blocks of 32 per wave (D = 32 NW NB), RB row blocks of 32
template <int NW, int NB, int RB>
struct PanelShape {
  static constexpr int D = 32 * NW * NB, CH = 32 * NW, ROWS = 32 * RB;
  static constexpr int kA = ROWS * D * 2, kH = ROWS * CH * 2, kStat = ROWS * NW * NB * 4;
  static constexpr int kRowX = D * 4;                                          // a row of the stream
  static constexpr int kHs = 2 * kH > 32 * kRowX ? 2 * kH : 32 * kRowX;        // both buffers of the hidden layer, or 32 rows of the stream
  // The stream waits in registers while FC2 is summed, but for these quads of a lane, which wait in LDS: there are not registers for all.
  static constexpr int kWait = RB * NB == 4 ? 2 : 0;
  static constexpr int kLds = kA + kHs + 2 * kStat + kWait * NW * 1024;
  static constexpr int PF = RB * NB == 1 ? 16 : 8;      // weight fragments in flight
  static constexpr int AF = RB == 1 ? 4 : RB == 2 ? 3 : 2;      // row fragments, the one in use included
};

template <int NW, int NB, int RB>
__global__ __launch_bounds__(NW * 64, NW / 4) void panel_block_kernel(PanelArgs g) {
  typedef PanelShape<NW, NB, RB> S;
  constexpr int D = S::D, CH = S::CH, ROWS = S::ROWS, PF = S::PF;
  constexpr int KD = D / 16, KC = CH / 16;             // k steps over the features and over a chunk
  constexpr int NG = NW * NB;                          // column groups of 32 a row has
  static_assert(KD % PF == 0 && (KC * NB) % PF == 0 && D % 128 == 0 && 4 * CH >= 2 * D, "units hold whole rings");
  extern __shared__ __align__(1024) unsigned char smem[];
  constexpr int sA = 0, sH = S::kA;                     // rows (attention output, then normalised stream), hidden layer twice
  float *const stat = reinterpret_cast<float *>(smem + S::kA + S::kHs);      // [2][ROWS][NG]

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int m0 = blockIdx.x * ROWS;

  // ---- rows of the attention output into LDS; rows past the end repeat the last one and are never stored
  {
    constexpr int CPR = D / 8, LOADS = ROWS * CPR / 64;
#pragma unroll
    for (int i = 0; i < (LOADS + NW - 1) / NW; ++i) {
      const int blk = wave + NW * i;
      if (LOADS % NW == 0 || blk < LOADS) {
        const int L = blk * 64 + lane, row = L / CPR, c = (L % CPR) ^ (row & 15);
        attn_dl_load16(g.a + static_cast<size_t>(min(m0 + row, g.M - 1)) * D + c * 8, smem + sA + blk * 1024);
      }
    }
  }

  // ---- weight stream: a ring of PF fragments.  One buffer covers the packed matrices that the launch reads; a unit is named by the
  // byte offset of the wave's first fragment in it, a scalar, to which a lane adds 16 bytes times its number.
  const __amdgpu_buffer_rsrc_t weights = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(g.w), 0, static_cast<int>(g.w_bytes), 0x00020000);
  const int lane16 = lane * 16;
  auto fragment = [&](int unit, int f) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(weights, lane16, unit + f * 1024, 0));
  };
  auto unit_at = [&](int matrix, int u, int frags) { return matrix + (u * NW + wave) * frags * 1024; };
  const int p_proj = unit_at(g.w_proj, 0, KD * NB);
  auto p_fc1 = [&](int c) { return unit_at(g.w_fc1, c, KD); };
  auto p_fc2 = [&](int c) { return unit_at(g.w_fc2, c, KC * NB); };
  auto p_qkv = [&](int p) { return unit_at(g.w_qkv, p, 3 * KD); };
  bf16x8 ring[PF];
#pragma unroll
  for (int i = 0; i < PF; ++i) ring[i] = fragment(p_proj, i);
  // everybody's LDS accesses done; the fragments in flight stay in flight (__syncthreads() would wait for them)
  auto sync = [&]() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };

  // LDS addresses are one register each: chunk 2 kk + hi of a row is at (its address for kk = 0) ^ 32 kk for the first eight steps and
  // 256 bytes further on for the next eight, the column quads q of a wave's 32 columns at (that of q = 0) ^ 16 q.  The empty
  // statement keeps the compiler from holding all of them, for every buffer, in registers across the units (it spills otherwise).
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)smem));
  auto lds = [](unsigned at, auto type) {
    return reinterpret_cast<__attribute__((address_space(3))) decltype(type) *>(at);
  };
  auto fresh_lane = [&]() {
    int l = lane;
    asm volatile("" : "+v"(l));
    return l;
  };
  auto read_base = [&](int buffer, int pitch) {
    const int l = fresh_lane(), r = l & 31;
    return lds0 + buffer + r * pitch + (((l >> 5) ^ (r & 15)) << 4);
  };
  auto write_base = [&](int buffer, int pitch, int block) {
    const int l = fresh_lane(), r = l & 31;
    return lds0 + buffer + r * pitch + ((block * 4 ^ (r & 15)) << 4) + (l >> 5) * 8;
  };

  // acc[i][j] += rows of block i (LDS from `rows` on, PITCH bytes a row) times the unit's fragments, from init() on where that is
  // not acc itself; `next`: the unit after it.  beside(f): vector work to go with the matrix instructions of fragment f.
  auto unit = [&](auto kk_c, auto nb_c, auto pitch_c, f32x16 (*acc)[decltype(nb_c)::value], auto init, int rows, int cur, int next, auto beside) {
    constexpr int KK = decltype(kk_c)::value, N = decltype(nb_c)::value, PITCH = decltype(pitch_c)::value, AF = S::AF;
    const unsigned r0 = read_base(rows, PITCH);
    bf16x8 af[AF][RB];
    auto fetch = [&](int kk) {
#pragma unroll
      for (int i = 0; i < RB; ++i) af[kk % AF][i] = *lds((r0 ^ (kk % 8 * 32)) + i * 32 * PITCH + kk / 8 * 256, bf16x8{});
    };
#pragma unroll
    for (int kk = 0; kk < AF - 1; ++kk) fetch(kk);
    each<KK>([&](auto kk_c) {
      constexpr int kk = decltype(kk_c)::value;
      if constexpr (kk + AF - 1 < KK) fetch(kk + AF - 1);
      each<N>([&](auto j_c) {
        constexpr int j = decltype(j_c)::value, f = kk * N + j;
        const bf16x8 w = ring[f % PF];
#pragma unroll
        for (int i = 0; i < RB; ++i)            // operands swapped: the block is C^T
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w, af[kk % AF][i], kk == 0 ? init(i, j) : acc[i][j], 0, 0, 0);
        ring[f % PF] = f + PF < KK * N ? fragment(cur, f + PF) : fragment(next, f + PF - KK * N);
        beside(std::integral_constant<int, f>{});
        if constexpr (!std::is_same<decltype(beside), Nothing>::value) {
#pragma unroll
          for (int i = 0; i < RB; ++i) {
            if (i == 0) __builtin_amdgcn_sched_group_barrier(0x100, RB, 0);      // the next step's row fragments are requested first
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                   // a matrix instruction,
            __builtin_amdgcn_sched_group_barrier(0x002, RB == 3 ? 10 : 13, 0);    // then its share of a piece of vector work
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  typedef std::integral_constant<int, KD> KDc;
  typedef std::integral_constant<int, KC> KCc;
  typedef std::integral_constant<int, 1> One;
  typedef std::integral_constant<int, NB> NBc;
  typedef std::integral_constant<int, 2 * D> PitchD;
  typedef std::integral_constant<int, 2 * CH> PitchC;

  // registers 4 q .. 4 q + 3 of a block: columns 8 q + 4 hi + 0..3 of row lane % 32 (hi = lane / 32)
  auto load4 = [](const float *p) { return *reinterpret_cast<const float4 *>(p); };
  auto load_quads = [&](const float *p) {      // of 32 columns from p on, in the order of an accumulator block
    f32x16 v;
    const int h4 = 4 * (fresh_lane() >> 5);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 f = load4(p + 8 * q + h4);
      v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
    }
    return v;
  };

  // x [RB][NB]: rows normalised into LDS (sA), ready behind the barrier that ends it
  auto layernorm = [&](const f32x16 (&x)[RB][NB], const float *gain, const float *bias, auto behind_first_barrier) {
    float mean[RB], rstd[RB];
    f32x16 ga, be;                               // of one column block, requested ahead
    auto request = [&](int j) {
      ga = load_quads(gain + (wave * NB + j) * 32);
      be = load_quads(bias + (wave * NB + j) * 32);
    };
    request(0);
    auto row_total = [&](float *box, const float (&part)[RB][NB]) {
      const int l = fresh_lane();
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          unsigned lo, up;
          lane_pair_exchange(__builtin_bit_cast(unsigned, part[i][j]), lo, up);
          if (l < 32) box[(i * 32 + l) * NG + wave * NB + j] = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, up);
        }
      sync();
    };
    auto tree = [&](const float *box, int i) {
      const float *p = box + (i * 32 + (fresh_lane() & 31)) * NG;
      float v[NG];
#pragma unroll
      for (int k = 0; k < NG; k += 4) {
        const float4 f = load4(p + k);
        v[k] = f.x; v[k + 1] = f.y; v[k + 2] = f.z; v[k + 3] = f.w;
      }
#pragma unroll
      for (int s = 1; s < NG; s *= 2)
#pragma unroll
        for (int k = 0; k + s < NG; k += 2 * s) v[k] += v[k + s];
      return v[0];
    };
    float part[RB][NB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        float s[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] = ln_sum4(x[i][j][4 * q], x[i][j][4 * q + 1], x[i][j][4 * q + 2], x[i][j][4 * q + 3]);
        part[i][j] = (s[0] + s[1]) + (s[2] + s[3]);
      }
    row_total(stat, part);
    behind_first_barrier();
#pragma unroll
    for (int i = 0; i < RB; ++i) mean[i] = tree(stat, i) / static_cast<float>(D);
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        float s[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
          s[q] = ln_square4(x[i][j][4 * q] - mean[i], x[i][j][4 * q + 1] - mean[i], x[i][j][4 * q + 2] - mean[i], x[i][j][4 * q + 3] - mean[i]);
        part[i][j] = (s[0] + s[1]) + (s[2] + s[3]);
      }
    row_total(stat + ROWS * NG, part);
#pragma unroll
    for (int i = 0; i < RB; ++i) rstd[i] = ln_rstd(tree(stat + ROWS * NG, i), static_cast<float>(D));
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const unsigned w0 = write_base(sA, 2 * D, wave * NB + j);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const f32x16 &v = x[i][j];
          u32x2 p;
          p[0] = pack2(ln_apply(v[4 * q], mean[i], rstd[i], ga[4 * q], be[4 * q]), ln_apply(v[4 * q + 1], mean[i], rstd[i], ga[4 * q + 1], be[4 * q + 1]));
          p[1] = pack2(ln_apply(v[4 * q + 2], mean[i], rstd[i], ga[4 * q + 2], be[4 * q + 2]), ln_apply(v[4 * q + 3], mean[i], rstd[i], ga[4 * q + 3], be[4 * q + 3]));
          *lds((w0 ^ (q * 16)) + i * 32 * (2 * D), u32x2{}) = p;
        }
      }
      if (j + 1 < NB) request(j + 1);
    }
    sync();
  };
  // ---- projection.  Rows of the stream come and go through LDS as fp32,
  // 16-byte chunk c of row r at c ^ (r & 15): in memory a wave moves whole lines.  Straight from and to the accumulator layout it
  // touches 32 lines an instruction, and at D = 256 the stores of 96 rows took 4.5 us of a panel's 43.
  constexpr int kRowX = S::kRowX, XPR = D / 4, XB = S::kHs / (32 * kRowX) < RB ? S::kHs / (32 * kRowX) : RB;      // row blocks at a time
  static_assert(XPR * 32 % (64 * NW) == 0 && ROWS * kRowX <= S::kA + S::kHs, "stream rows in LDS");
  auto x_at = [&](int base, int j) {             // chunk of quad 0 of the lane's row; quad q at ^ 32 q
    const int l = fresh_lane(), r = l & 31;
    return lds0 + base + r * kRowX + ((((wave * NB + j) * 8 + (l >> 5)) ^ (r & 15)) << 4);
  };
  f32x16 x[RB][NB];
#pragma unroll
  for (int i0 = 0; i0 < RB; i0 += XB) {
    if (i0 > 0) sync();
#pragma unroll
    for (int k = 0; k < XB * 32 * XPR / (64 * NW); ++k) {
      const int blk = wave + NW * k, L = blk * 64 + lane, row = L / XPR, c = (L % XPR) ^ (row & 15);
      const int m = min(m0 + i0 * 32 + row, g.M - 1);
      const size_t src = g.res_map ? static_cast<size_t>(m / g.res_out) * g.res_in + g.res_map[m % g.res_out] : static_cast<size_t>(m);
      attn_dl_load16(reinterpret_cast<const bf16_t *>(g.res + src * D + c * 4), smem + sH + blk * 1024);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
    sync();
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const unsigned at = x_at(sH, j);
#pragma unroll
      for (int i = 0; i < XB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 v = *lds((at ^ (q * 32)) + i * 32 * kRowX, f32x4{});
          f32x16 &d = x[i0 + i][j];
          d[4 * q] = v[0]; d[4 * q + 1] = v[1]; d[4 * q + 2] = v[2]; d[4 * q + 3] = v[3];
        }
    }
  }
  f32x16 sum[RB][NB];
  auto from_sum = [&](int i, int j) { return sum[i][j]; };
  auto from_zero = [](int, int) { return f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}; };
  // x <- (sum + bias) + x, the order of the products' epilogues
  auto add_to_stream = [&](const float *bias) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const f32x16 b = load_quads(bias + (wave * NB + j) * 32);
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) x[i][j][r] = (sum[i][j][r] + b[r]) + x[i][j][r];
    }
  };
  unit(KDc{}, NBc{}, PitchD{}, sum, from_zero, sA, p_proj, p_fc1(0), Nothing{});
  add_to_stream(g.b_proj);
  __builtin_amdgcn_sched_barrier(0);             // registers: nothing of what follows is requested before the LayerNorm is done
  layernorm(x, g.ln2_g, g.ln2_b, []() {});       // its first barrier: nobody reads the attention output any more
  __builtin_amdgcn_sched_barrier(0);
  auto waiting = [&](int k) { return lds(lds0 + S::kLds - (k + 1) * NW * 1024 + (wave * 64 + fresh_lane()) * 16, f32x4{}); };
#pragma unroll
  for (int k = 0; k < S::kWait; ++k) {
    const f32x16 &v = x[RB - 1][NB - 1];
    *waiting(k) = f32x4{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
  }

  // ---- feed-forward layer.  GELU of chunk c runs beside the matrix instructions of FC2 of chunk c - 1 and FC1 of chunk c + 1, two
  // values at a time; then a barrier, and chunk c is whole.
  const int chunks = g.R / CH;
  f32x16 ha[RB][1], hb[RB][1];                  // FC1 of even and odd chunks
  // the bias of the column quad that GELU takes and of the one after it: quad q at 4 (q % 2)
  typedef __attribute__((ext_vector_type(8))) float f32x8;
  const float *const b_fc1 = g.b_fc1 + wave * 32;
  f32x8 bias;
  auto fetch_bias = [&](int c, int q) {
    const float4 f = load4(b_fc1 + c * CH + 8 * q + 4 * (fresh_lane() >> 5));
    const int k = 4 * (q & 1);
    bias[k] = f.x; bias[k + 1] = f.y; bias[k + 2] = f.z; bias[k + 3] = f.w;
  };
  fetch_bias(0, 0);
  fetch_bias(0, 1);
#pragma unroll
  for (int i = 0; i < RB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) sum[i][j] = from_zero(i, j);
  constexpr int PIECES = 8 * RB, F1 = KD, F2 = KC * NB;      // pieces of two values; fragments of the units
  uint32_t low = 0;
  auto gelu_piece = [&](const f32x16 (&h)[RB][1], unsigned w0, int c, auto n_c) {
    constexpr int n = decltype(n_c)::value, q = n / (2 * RB), i = n / 2 % RB, e = 4 * q + 2 * (n & 1), k = e & 7;
    const uint32_t p = pack2(gelu_erf_fast(h[i][0][e] + bias[k]), gelu_erf_fast(h[i][0][e + 1] + bias[k + 1]));
    if constexpr (n & 1) *lds((w0 ^ (q * 16)) + i * 32 * (2 * CH), u32x2{}) = u32x2{low, p};
    else low = p;
    if constexpr (n % (2 * RB) == 2 * RB - 1) fetch_bias(q < 2 ? c : min(c + 1, chunks - 1), (q + 2) % 4);
  };
  // the pieces of chunk c that go with fragment F of OF
  auto gelu_beside = [&](const f32x16 (&h)[RB][1], unsigned w0, int c, auto f_c, auto of_c) {
    constexpr int F = decltype(f_c)::value, OF = decltype(of_c)::value, first = F * PIECES / OF;
    each<(F + 1) * PIECES / OF - first>([&](auto k) { gelu_piece(h, w0, c, std::integral_constant<int, first + decltype(k)::value>{}); });
  };
  typedef std::integral_constant<int, F1> OfF1;
  typedef std::integral_constant<int, F2> OfF2;
  typedef std::integral_constant<int, F1 + F2> OfBoth;
  auto buffer = [&](int c) { return sH + (c & 1) * S::kH; };
  auto fc1 = [&](int c, f32x16 (&h)[RB][1], int next, auto beside) {
    unit(KDc{}, One{}, PitchD{}, h, from_zero, sA, p_fc1(c), next, beside);
  };
  auto fc2 = [&](int c, int next, auto beside) { unit(KCc{}, NBc{}, PitchC{}, sum, from_sum, buffer(c), p_fc2(c), next, beside); };
  const int after = g.qkv ? p_qkv(0) : p_proj;      // no next block: fetched, not used
  // FC2 of chunk c - 1, GELU of chunk c (in h), FC1 of chunk c + 1 (into other)
  auto interval = [&](int c, const f32x16 (&h)[RB][1], f32x16 (&other)[RB][1]) {
    const unsigned w0 = write_base(buffer(c), 2 * CH, wave);
    fc2(c - 1, p_fc1(c + 1), [&](auto f) { gelu_beside(h, w0, c, f, OfBoth{}); });
    fc1(c + 1, other, p_fc2(c), [&](auto f) { gelu_beside(h, w0, c, std::integral_constant<int, F2 + decltype(f)::value>{}, OfBoth{}); });
    sync();
  };
  auto last = [&](const f32x16 (&h)[RB][1]) {
    const int c = chunks - 1, w0 = write_base(buffer(c), 2 * CH, wave);
    fc2(c - 1, p_fc2(c), [&](auto f) { gelu_beside(h, w0, c, f, OfF2{}); });
    sync();
  };
  fc1(0, ha, p_fc1(1), Nothing{});
  {
    const unsigned w0 = write_base(buffer(0), 2 * CH, wave);
    fc1(1, hb, p_fc2(0), [&](auto f) { gelu_beside(ha, w0, 0, f, OfF1{}); });
    sync();
  }
#pragma unroll 1
  for (int c = 1; c + 2 < chunks; c += 2) {      // an even number of chunks
    interval(c, hb, ha);
    interval(c + 1, ha, hb);
  }
  last(hb);
  fc2(chunks - 1, after, Nothing{});
#pragma unroll
  for (int k = 0; k < S::kWait; ++k) {
    const f32x4 v = *waiting(k);
    f32x16 &d = x[RB - 1][NB - 1];
    d[4 * k] = v[0]; d[4 * k + 1] = v[1]; d[4 * k + 2] = v[2]; d[4 * k + 3] = v[3];
  }
  add_to_stream(g.b_fc2);
  // the stream's rows to LDS (nothing else lies there any more once everybody has left FC2) and from there to memory
  auto x_to_lds = [&]() {
    sync();
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const unsigned at = x_at(0, j);
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x16 &v = x[i][j];
          *lds((at ^ (q * 32)) + i * 32 * kRowX, f32x4{}) = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
        }
    }
  };
  auto x_to_memory = [&]() {
#pragma unroll
    for (int k = 0; k < ROWS * XPR / (64 * NW); ++k) {
      const int L = (k * NW + wave) * 64 + fresh_lane(), r = L / XPR, c = L % XPR;
      const f32x4 v = *lds(lds0 + r * kRowX + ((c ^ (r & 15)) << 4), f32x4{});
      if (m0 + r < g.M) *reinterpret_cast<f32x4 *>(g.x + static_cast<size_t>(m0 + r) * D + c * 4) = v;
    }
  };
  x_to_lds();
  if (!g.qkv) {
    sync();
    x_to_memory();
    return;
  }

  // ---- the next block's LayerNorm and qkv, CH columns at a time through the hidden layer's buffers: the results of unit u go to LDS
  // beside the matrix instructions of unit u + 1
  layernorm(x, g.ln1_g, g.ln1_b, x_to_memory);
  constexpr int PASSES = D / CH;
  f32x16 h[RB][3];
  auto to_lds = [&](int u, int j, int base) {
    const float sc = u * CH + wave * 32 < D ? g.qscale : 1.0f;
    const f32x16 b = load_quads(g.b_qkv + u * CH + wave * 32);
    const unsigned w0 = write_base(base, 2 * CH, wave);
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const f32x16 &v = h[i][j];
        u32x2 p;
        p[0] = pack2((v[4 * q] + b[4 * q]) * sc, (v[4 * q + 1] + b[4 * q + 1]) * sc);
        p[1] = pack2((v[4 * q + 2] + b[4 * q + 2]) * sc, (v[4 * q + 3] + b[4 * q + 3]) * sc);
        *lds((w0 ^ (q * 16)) + i * 32 * (2 * CH), u32x2{}) = p;
      }
  };
  auto to_memory = [&](int u, int base) {
    constexpr int CPR = CH / 8;
#pragma unroll
    for (int it = 0; it < ROWS * CPR / (NW * 64); ++it) {
      const int L = (it * NW + wave) * 64 + fresh_lane(), r = L / CPR, c = L % CPR;
      const u32x4 v = *lds(lds0 + base + r * (2 * CH) + ((c ^ (r & 15)) << 4), u32x4{});
      if (m0 + r < g.M) *reinterpret_cast<u32x4 *>(g.qkv + static_cast<size_t>(m0 + r) * (3 * D) + u * CH + c * 8) = v;
    }
  };
#pragma unroll 1
  for (int p = 0; p < PASSES; ++p) {            // 3 CH columns
    unit(KDc{}, std::integral_constant<int, 3>{}, PitchD{}, h, from_zero, sA, p_qkv(p), p + 1 < PASSES ? p_qkv(p + 1) : p_proj, Nothing{});
    if (p > 0) sync();                          // the pass before has left the buffers
    to_lds(3 * p, 0, sH);
    to_lds(3 * p + 1, 1, sH + S::kH);
    sync();
    to_memory(3 * p, sH);
    to_memory(3 * p + 1, sH + S::kH);
    const int third = p + 1 < PASSES ? sH : sA; // nobody reads the normalised rows behind the last pass's barrier
    if (p + 1 < PASSES) sync();
    to_lds(3 * p + 2, 2, third);
    sync();
    to_memory(3 * p + 2, third);
  }
}

// ------------------------------------------------------------------ packing
// w [N, K] -> fragments in the order of the panel kernel: unit (a group of 32 nw nb columns, or of kk steps of 16 k), wave,
// step, column block of the wave, then 64 lanes x 8 values.  A wave's nb column blocks lie next to each other, or `spread`
// (qkv) nw blocks apart.
__global__ __launch_bounds__(256) void panel_pack_kernel(const bf16_t *w, bf16_t *out, int N, int K, int nw, int nb, int kk, int spread) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= static_cast<int64_t>(N) * K / 8) return;
  const int lane = static_cast<int>(i % 64);
  int64_t f = i / 64;
  const int j = static_cast<int>(f % nb);
  f /= nb;
  const int step = static_cast<int>(f % kk);
  f /= kk;
  const int wave = static_cast<int>(f % nw), u = static_cast<int>(f / nw);
  const int kg = K / (16 * kk);                 // units along k (else along the columns)
  const int block = (kg > 1 ? 0 : u) * nw * nb + (spread ? j * nw + wave : wave * nb + j);
  const int n = block * 32 + (lane & 31);
  const int k = ((kg > 1 ? u : 0) * kk + step) * 16 + (lane >> 5) * 8;
  *reinterpret_cast<u32x4 *>(out + i * 8) = *reinterpret_cast<const u32x4 *>(w + static_cast<size_t>(n) * K + k);
}

static int g_panel_cus = 0;

template <int NW, int NB, int RB>
static hipError_t panel_attr() {
  return hipFuncSetAttribute(reinterpret_cast<const void *>(&panel_block_kernel<NW, NB, RB>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             PanelShape<NW, NB, RB>::kLds);
}

hipError_t panel_init() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if ((e = hipDeviceGetAttribute(&g_panel_cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return e;
  if ((e = panel_attr<8, 1, 1>()) != hipSuccess || (e = panel_attr<8, 1, 2>()) != hipSuccess || (e = panel_attr<8, 1, 3>()) != hipSuccess) return e;
  if ((e = panel_attr<8, 2, 1>()) != hipSuccess || (e = panel_attr<8, 2, 2>()) != hipSuccess) return e;
  return hipSuccess;
}

bool panel_used(const reslim_ctx *c, int64_t rows, const void *stream) {
  return c->d_panel_w && !gemm_pinned() && rows >= panel_rows_from(c->cfg.embed_dim, c->R) && (reinterpret_cast<uintptr_t>(stream) & 15) == 0;
}

bool panel_takes(const reslim_ctx *c) { return c->cfg.dtype == RESLIM_BF16 && panel_width(c->cfg.embed_dim) && c->R % 512 == 0 && c->cfg.mlp_ratio <= 256; }

// What one launch reads lies together: a layer's three matrices, then the qkv of the layer after it.  The first layer's qkv has no
// launch that would read it.
static size_t panel_layer_elems(const reslim_ctx *c) { return static_cast<size_t>(c->cfg.embed_dim) * (4 * c->cfg.embed_dim + 2 * c->R); }
static size_t panel_qkv_elems(const reslim_ctx *c) { return static_cast<size_t>(3) * c->cfg.embed_dim * c->cfg.embed_dim; }
size_t panel_elems(const reslim_ctx *c) { return panel_layer_elems(c) * c->cfg.depth - panel_qkv_elems(c); }

hipError_t panel_pack(const reslim_ctx *c, int layer, bf16_t *dst, hipStream_t st) {
  const LayerWeights &lw = c->layers[layer];
  dst += panel_layer_elems(c) * layer;
  const int D = c->cfg.embed_dim, R = c->R, nw = 8, nb = D / (32 * nw), ch = 32 * nw;
  const bool last = layer + 1 == c->cfg.depth;
  // one after the other, as launch_panel_block() counts
  const struct { const void *src; int N, K, nb, kk, spread; } todo[4] = {
      {lw.w_proj, D, D, nb, D / 16, 0}, {lw.w_fc1, R, D, 1, D / 16, 0}, {lw.w_fc2, D, R, nb, ch / 16, 0},
      {last ? nullptr : c->layers[layer + 1].w_qkv, 3 * D, D, 3, D / 16, 1}};
  for (auto &td : todo) {
    if (!td.src) continue;
    const int64_t n = static_cast<int64_t>(td.N) * td.K;
    panel_pack_kernel<<<dim3(static_cast<unsigned>((n / 8 + 255) / 256)), dim3(256), 0, st>>>(static_cast<const bf16_t *>(td.src), dst, td.N, td.K,
                                                                                             nw, td.nb, td.kk, td.spread);
    dst += n;
  }
  return hipGetLastError();
}

hipError_t launch_panel_block(const reslim_ctx *c, int layer, const void *a, const float *res, const ResRowMap *res_map, float *x, void *qkv_next,
                              int M, hipStream_t st) {
  if (M <= 0 || (qkv_next && layer + 1 >= c->cfg.depth)) return hipErrorInvalidValue;
  const LayerWeights &lw = c->layers[layer];
  const LayerWeights &nx = c->layers[qkv_next ? layer + 1 : layer];
  PanelArgs g;
  g.a = static_cast<const bf16_t *>(a);
  g.res = res;
  g.res_map = res_map ? res_map->map : nullptr;
  g.res_out = res_map ? res_map->rows_out : 1;
  g.res_in = res_map ? res_map->rows_in : 1;
  g.x = x;
  g.qkv = static_cast<bf16_t *>(qkv_next);
  const size_t D = c->cfg.embed_dim, R = c->R, es = sizeof(bf16_t);
  g.w = c->d_panel_w + panel_layer_elems(c) * layer;
  g.w_bytes = static_cast<unsigned>((panel_layer_elems(c) - (qkv_next ? 0 : panel_qkv_elems(c))) * es);
  g.w_proj = 0;
  g.w_fc1 = static_cast<int>(D * D * es);
  g.w_fc2 = static_cast<int>((D * D + R * D) * es);
  g.w_qkv = static_cast<int>((D * D + 2 * R * D) * es);
  g.b_proj = lw.b_proj; g.b_fc1 = lw.b_fc1; g.b_fc2 = lw.b_fc2; g.b_qkv = nx.b_qkv;
  g.ln2_g = lw.ln2_g; g.ln2_b = lw.ln2_b; g.ln1_g = nx.ln1_g; g.ln1_b = nx.ln1_b;
  g.M = M;
  g.R = c->R;
  g.qscale = 1.4426950408889634f / sqrtf(static_cast<float>(c->dh));
  const int rb = panel_row_blocks(M, g_panel_cus, D == 256 ? 3 : 2);
  const dim3 grid((M + 32 * rb - 1) / (32 * rb)), blk(512);
#define RESLIM_PANEL(NB, RB) panel_block_kernel<8, NB, RB><<<grid, blk, PanelShape<8, NB, RB>::kLds, st>>>(g)
  if (D == 256) {
    if (rb == 1) RESLIM_PANEL(1, 1);
    else if (rb == 2) RESLIM_PANEL(1, 2);
    else RESLIM_PANEL(1, 3);
  } else {
    if (rb == 1) RESLIM_PANEL(2, 1);
    else RESLIM_PANEL(2, 2);
  }
#undef RESLIM_PANEL
  return hipGetLastError();
}

}  // namespace reslim
