// Dense contractions of the transformer block (ORBIT-2 Sec. 3 / 4.1: the QKV,
// projection and feed-forward maps, the aggregation's output map and the decoder's
// linear projection):   C[M, N] (+)= A[M, K] * W[N, K]^T + bias, fused epilogues.
//
// bf16 path: gfx950 MFMA 32x32x16 (bf16 in, fp32 accumulate), three kernels of which
// gemm_choose (gemm_plan.h) takes one by estimated time: the persistent ones of 256 x 256 and
// 128 x 256 tiles (gemm_pp.inc) and gemm_bf16_kernel with one 128 x 128 tile per
// work-group.  That one stages BM x BK and BN x BK operand slabs through LDS (rows
// padded by 16 B so the 16-byte fragment reads of 16 consecutive rows fall in
// distinct bank groups), the next slab prefetched into registers while the current
// one feeds the matrix cores.  Its work-groups are renumbered so that each XCD
// (private L2) receives a contiguous run of tiles, and inside a run tiles are ordered
// in bands of GROUP_M row-tiles so concurrently resident tiles share A and W slabs.
// fp32 path: MFMA 32x32x2 in fp32, operands straight from global memory.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "gelu.h"
#include "gemm_cursor.h"
#include "gemm_plan.h"

namespace reslim {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

struct GemmArgs {
  const void *A;
  const void *W;
  const float *bias;
  void *out;
  const float *tab;
  int ldo, tab_rows;
  int M, N, K;
  int grid_m, grid_n;
  float qscale;   // EPI_BIAS_QSCALE_ACT: factor applied to output columns n < qcols
  int qcols;
  int col_fast;            // one-tile-per-work-group kernel: tile order inside a band
  const void *aux;         // EPI_BIAS_RES_F32: skip input (fp32), layout of out unless res_map is set
  const int32_t *res_map;  // EPI_BIAS_RES_F32, optional: output row b*res_out + r reads skip row b*res_in + res_map[r]
  int res_out;
  int64_t res_in;
  void *out2;              // EPI_BIAS_ACT_GELU2: second output (act), layout of out
  // fp32 kernel with LayerNorm in front: gain and bias; rows of A through a map (see ResRowMap) where it is set
  const float *ln_g, *ln_b;
  const int32_t *a_map;
  int a_out;
  int64_t a_in;
};


__device__ __forceinline__ float gelu_erf(float x) {
  return 0.5f * x * (1.0f + erff(x * 0.70710678118654752440f));
}

// Every epilogue runs with the MFMA operand roles swapped: the accumulator block is
// then C^T, a lane holds one output row (lane % 32) and four consecutive columns per
// register quad.  All outputs go through a 4 KB staging area of the wave in LDS, bf16
// ones 32 rows x 64 columns at a time, fp32 ones 32 x 32, so that a store instruction
// writes eight complete 128-byte row segments (16 bytes per lane) instead of 32 or 64
// partial ones; no barrier is involved, the LDS operations of one wave execute in order.
template <int EPI>
__device__ __host__ constexpr bool epi_act_out() {
  return EPI == EPI_BIAS_ACT || EPI == EPI_BIAS_QSCALE_ACT || EPI == EPI_BIAS_GELU_ACT || EPI == EPI_BIAS_ACT_GELU2;
}
constexpr int kEpiStageBytes = 4096;    // per wave

// one value of a bf16-output epilogue (v already carries the bias); sc: the factor of the value's
// block of 32 columns (EPI_BIAS_QSCALE_ACT: qcols is a multiple of 32, so a block is scaled as a
// whole and the factor is one scalar per block, not a register per column)
template <int EPI, bool SECOND>
__device__ __forceinline__ float epi_act_value(float v, float sc) {
  if constexpr (EPI == EPI_BIAS_QSCALE_ACT) return v * sc;
  if constexpr (EPI == EPI_BIAS_GELU_ACT || (EPI == EPI_BIAS_ACT_GELU2 && SECOND)) return gelu_erf_fast(v);
  return v;
}

// Rows m_first .. m_first + 31, columns n_first .. n_first + 63 (two accumulator
// blocks side by side) of a bf16 output; bias[jj][q] holds the four bias values of
// this lane's column quad.  Staging layout: row r at 128 r bytes, its 16-byte chunk c at position c ^ ((r >> 1) & 7), and the two 8-byte halves of a
// chunk exchanged where r >= 16: with that the 8-byte writes of 32 lanes (32 rows,
// one column quad) and the 16-byte reads of 16 lanes (two rows) each touch every
// bank once.  N is a multiple of 8, so a 16-byte piece is inside the row or not at all.
template <int EPI, bool SECOND, bool GUARD>
__device__ __forceinline__ void epilogue_act_stage(const GemmArgs &g, const f32x16 *blk, const float4 (*bias)[4],
                                                   int m_first, int n_first, int lane, unsigned char *stg) {
  const int l32 = lane & 31, hi = lane >> 5;
  bf16_t *out = static_cast<bf16_t *>(SECOND ? g.out2 : g.out);
  unsigned char *wrow = stg + l32 * 128 + ((hi ^ (l32 >> 4)) << 3);
  const int wsw = (l32 >> 1) & 7;
#pragma unroll
  for (int jj = 0; jj < 2; ++jj) {
    const float sc = (EPI == EPI_BIAS_QSCALE_ACT && n_first + jj * 32 < g.qcols) ? g.qscale : 1.0f;   // uniform
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 b = bias[jj][q];
      u32x2 pk;
      pk[0] = pack2(epi_act_value<EPI, SECOND>(blk[jj][4 * q] + b.x, sc), epi_act_value<EPI, SECOND>(blk[jj][4 * q + 1] + b.y, sc));
      pk[1] = pack2(epi_act_value<EPI, SECOND>(blk[jj][4 * q + 2] + b.z, sc), epi_act_value<EPI, SECOND>(blk[jj][4 * q + 3] + b.w, sc));
      *reinterpret_cast<u32x2 *>(wrow + (((jj * 4 + q) ^ wsw) << 4)) = pk;
    }
  }
  constexpr int LPR = 8, RPI = 64 / LPR;           // read back row-major: lanes per row, rows per instruction
  const int c = lane % LPR, rr = lane / LPR;
  const int n = n_first + c * 8;
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int r = it * RPI + rr;
    u32x4 v = *reinterpret_cast<const u32x4 *>(stg + r * 128 + ((c ^ ((r >> 1) & 7)) << 4));
    if (it * RPI >= 16) v = u32x4{v[2], v[3], v[0], v[1]};
    const int m = m_first + r;
    if (!GUARD || (m < g.M && n < g.N)) *reinterpret_cast<u32x4 *>(out + static_cast<size_t>(m) * g.ldo + n) = v;
  }
  __builtin_amdgcn_sched_barrier(0);   // keeps the next block's arithmetic from being hoisted over this one (registers)
}

// fp32 outputs: rows m_base .. m_base + 32 MI - 1, columns n_base .. n_base + 32 NI - 1, one 32 x 32 block at a time
// through the wave's 4 KB of LDS (row r at 128 r bytes, its 16-byte chunk c at c ^ ((r >> 1) & 7): the column quads of
// 16 rows and the chunks of two rows both fall into 16 different bank groups).  Eight lanes then hold a row's 128
// bytes, so a load or store instruction moves eight whole lines; straight from the accumulator layout it touches 32
// lines, 32 bytes of each, and the address path of the compute unit, not the memory, sets the pace (403,200 x 1024
// outputs with skip connection: 0.775 -> 0.648 ms on top of a 64-deep product, 1.24 -> 1.00 of a 1024-deep one).  The skip input (or the table) of the next DEPTH blocks is
// requested ahead of the block at hand.  The skip input may be the output itself: a lane reads what it writes.
template <int EPI, bool GUARD, int MI, int NI, int DEPTH>
__device__ __forceinline__ void epilogue_f32(const GemmArgs &g, const f32x16 (&acc)[MI][NI], int m_base, int n_base, int lane,
                                             unsigned char *stg) {
  constexpr bool kAdd = EPI != EPI_BIAS_F32, kTab = EPI == EPI_BIAS_TAB_F32;
  const int l32 = lane & 31, hi = lane >> 5, lr = lane >> 3, lc = lane & 7;
  auto col = [&](int j) { return GUARD ? min(n_base + j * 32 + lc * 4, g.N - 4) : n_base + j * 32 + lc * 4; };
  const float *src = kTab ? g.tab : EPI == EPI_BIAS_RES_F32 ? static_cast<const float *>(g.aux) : static_cast<const float *>(g.out);
  const bool mapped = EPI == EPI_BIAS_RES_F32 && g.res_map;      // uniform
  float4 x[DEPTH][4];
  auto fetch = [&](int b) {
    if constexpr (kAdd) {
      const int i = b / NI, j = b % NI;
#pragma unroll
      for (int it = 0; it < 4; ++it) {
        const int mu = m_base + i * 32 + it * 8;                 // uniform
        const int m = GUARD ? min(mu + lr, g.M - 1) : mu + lr;
        const float *p;
        if constexpr (kTab) {
          p = src + static_cast<size_t>(m % g.tab_rows) * g.N + col(j);
        } else if (mapped) {
          p = src + (static_cast<size_t>(m / g.res_out) * g.res_in + g.res_map[m % g.res_out]) * g.ldo + col(j);
        } else if constexpr (GUARD) {
          p = src + static_cast<size_t>(m) * g.ldo + col(j);
        } else {                                                 // uniform base, one 32-bit offset per lane
          p = src + static_cast<size_t>(mu) * g.ldo + n_base + j * 32 + static_cast<unsigned>(lr * g.ldo + lc * 4);
        }
        x[b % DEPTH][it] = *reinterpret_cast<const float4 *>(p);
      }
    }
  };
#pragma unroll
  for (int b = 0; b < DEPTH && b < MI * NI; ++b) fetch(b);
  float4 bias[NI];
  if constexpr (!kTab) {
#pragma unroll
    for (int j = 0; j < NI; ++j) bias[j] = *reinterpret_cast<const float4 *>(g.bias + col(j));
  }
  unsigned char *wrow = stg + l32 * 128;
  const int wsw = (l32 >> 1) & 7;
#pragma unroll
  for (int b = 0; b < MI * NI; ++b) {
    const int i = b / NI, j = b % NI;
    const f32x16 &a = acc[i][j];
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4 *>(wrow + (((2 * q + hi) ^ wsw) << 4)) = make_float4(a[4 * q], a[4 * q + 1], a[4 * q + 2], a[4 * q + 3]);
#pragma unroll
    for (int it = 0; it < 4; ++it) {
      const int r = it * 8 + lr;
      float4 v = *reinterpret_cast<const float4 *>(stg + r * 128 + ((lc ^ ((r >> 1) & 7)) << 4));
      if constexpr (!kTab) { v.x += bias[j].x; v.y += bias[j].y; v.z += bias[j].z; v.w += bias[j].w; }
      if constexpr (kAdd) {
        const float4 s = x[b % DEPTH][it];
        v.x += s.x; v.y += s.y; v.z += s.z; v.w += s.w;
      }
      const int mu = m_base + i * 32 + it * 8;
      float *o = static_cast<float *>(g.out) + static_cast<size_t>(mu) * g.ldo + n_base + j * 32 + static_cast<unsigned>(lr * g.ldo + lc * 4);
      if (!GUARD || (mu + lr < g.M && n_base + j * 32 + lc * 4 < g.N)) *reinterpret_cast<float4 *>(o) = v;
    }
    __builtin_amdgcn_sched_barrier(0);
    if (b + DEPTH < MI * NI) fetch(b + DEPTH);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// bf16 outputs: column blocks are taken two at a time, the bias of the lane's eight column quads is fetched once per pair.
template <int EPI, bool GUARD, int MI, int NI>
__device__ __forceinline__ void epilogue_act(const GemmArgs &g, const f32x16 (&acc)[MI][NI], int m_base, int n_base, int lane,
                                             unsigned char *stg) {
  const int hi = lane >> 5;
  static_assert(NI % 2 == 0, "column blocks come in pairs");
#pragma unroll
  for (int j0 = 0; j0 < NI; j0 += 2) {
    float4 bias[2][4];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n = n_base + (j0 + jj) * 32 + 8 * q + 4 * hi;
        bias[jj][q] = *reinterpret_cast<const float4 *>(g.bias + (GUARD ? min(n, g.N - 4) : n));
      }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      epilogue_act_stage<EPI, false, GUARD>(g, &acc[i][j0], bias, m_base + i * 32, n_base + j0 * 32, lane, stg);
      if constexpr (EPI == EPI_BIAS_ACT_GELU2) {
        // the second output adds the bias again: without this the compiler keeps the biased values of a whole block and spills
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int q = 0; q < 4; ++q) asm volatile("" : "+v"(bias[jj][q].x), "+v"(bias[jj][q].y), "+v"(bias[jj][q].z), "+v"(bias[jj][q].w));
        epilogue_act_stage<EPI, true, GUARD>(g, &acc[i][j0], bias, m_base + i * 32, n_base + j0 * 32, lane, stg);
      }
    }
  }
}

// GUARD = false: the wave's part of the tile lies inside the output (the common case, decided per wave): no bounds
// test anywhere.  GUARD = true: rows past M and column quads past N compute on clamped (valid) addresses and skip only
// the store.  N is a multiple of 8: quads are whole or absent.  stg: this wave's kEpiStageBytes of LDS.
template <int EPI, bool GUARD, int MI, int NI>
__device__ __forceinline__ void epilogue_wave(const GemmArgs &g, const f32x16 (&acc)[MI][NI], int m_base, int n_base, int lane,
                                              unsigned char *stg) {
  if constexpr (epi_act_out<EPI>()) epilogue_act<EPI, GUARD, MI, NI>(g, acc, m_base, n_base, lane, stg);
  else epilogue_f32<EPI, GUARD, MI, NI, EPI == EPI_BIAS_RES_F32 ? 2 : 3>(g, acc, m_base, n_base, lane, stg);
}

// tile id seen by the hardware dispatcher -> tile id in XCD-contiguous order
__device__ __forceinline__ int xcd_remap(int pid, int total) {
  constexpr int NXCD = 8;
  const int x = pid % NXCD, local = pid / NXCD;
  const int q = total / NXCD, r = total % NXCD;
  return x * q + (x < r ? x : r) + local;
}

template <int BM, int BN, int BK, int WM, int WN, int NBUF, int MINW, int EPI>
__global__ __launch_bounds__(WM * WN * 64, MINW) void gemm_bf16_kernel(GemmArgs g) {
  constexpr int NT = WM * WN * 64;
  constexpr int PITCH = BK + 8;           // bf16 elements per LDS row
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int MI = TM / 32, NI = TN / 32;
  constexpr int KC = BK / 8;              // 16-byte chunks per slab row
  constexpr int CA = BM * KC / NT, CB = BN * KC / NT;
  static_assert(BM * KC % NT == 0 && BN * KC % NT == 0, "slab must split evenly over threads");
  static_assert(TM % 32 == 0 && TN % 32 == 0 && BK % 16 == 0, "MFMA tiling");
  constexpr int GROUP_M = 8;

  extern __shared__ __align__(16) unsigned char smem[];
  bf16_t *As = reinterpret_cast<bf16_t *>(smem);        // [NBUF][BM][PITCH]
  bf16_t *Bs = As + NBUF * BM * PITCH;                   // [NBUF][BN][PITCH]

  const int total = g.grid_m * g.grid_n;
  int pid = xcd_remap(blockIdx.x, total);
  const int band = GROUP_M * g.grid_n;
  const int band_id = pid / band;
  const int first_m = band_id * GROUP_M;
  const int band_rows = min(g.grid_m - first_m, GROUP_M);
  // inside a band: rows fastest by default; columns fastest (the tiles that share an
  // A panel are consecutive work-groups) when the host asks for it
  const int tile_m = g.col_fast ? first_m + (pid % band) / g.grid_n : first_m + (pid % band) % band_rows;
  const int tile_n = g.col_fast ? (pid % band) % g.grid_n : (pid % band) / band_rows;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const int t = threadIdx.x;
  const int lane = t & 63, wave = t >> 6;
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, hi = lane >> 5;

  const bf16_t *A = static_cast<const bf16_t *>(g.A);
  const bf16_t *W = static_cast<const bf16_t *>(g.W);
  const int K = g.K;

  // per-thread global source rows (clamped: rows past the edge read valid memory,
  // their results are never stored)
  const bf16_t *a_src[CA];
  const bf16_t *b_src[CB];
  int a_dst[CA], b_dst[CB];
#pragma unroll
  for (int i = 0; i < CA; ++i) {
    const int c = t + i * NT, row = c / KC, kc = c % KC;
    const int gm = min(m0 + row, g.M - 1);
    a_src[i] = A + static_cast<size_t>(gm) * K + kc * 8;
    a_dst[i] = row * PITCH + kc * 8;
  }
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    const int c = t + i * NT, row = c / KC, kc = c % KC;
    const int gn = min(n0 + row, g.N - 1);
    b_src[i] = W + static_cast<size_t>(gn) * K + kc * 8;
    b_dst[i] = row * PITCH + kc * 8;
  }

  u32x4 ra[CA], rb[CB];
  auto load_global = [&](int k0) {
#pragma unroll
    for (int i = 0; i < CA; ++i) ra[i] = *reinterpret_cast<const u32x4 *>(a_src[i] + k0);
#pragma unroll
    for (int i = 0; i < CB; ++i) rb[i] = *reinterpret_cast<const u32x4 *>(b_src[i] + k0);
  };
  auto store_lds = [&](int buf) {
    bf16_t *as = As + buf * BM * PITCH;
    bf16_t *bs = Bs + buf * BN * PITCH;
#pragma unroll
    for (int i = 0; i < CA; ++i) *reinterpret_cast<u32x4 *>(as + a_dst[i]) = ra[i];
#pragma unroll
    for (int i = 0; i < CB; ++i) *reinterpret_cast<u32x4 *>(bs + b_dst[i]) = rb[i];
  };

  f32x16 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int nk = K / BK;
  load_global(0);
  if constexpr (NBUF == 2) {
    store_lds(0);
    __syncthreads();
  }

  const int a_frag = (wm * TM + l32) * PITCH + hi * 8;
  const int b_frag = (wn * TN + l32) * PITCH + hi * 8;

  // NBUF == 2: one barrier per slab, the next slab is written to the other buffer
  // after this one has been consumed.  NBUF == 1: half the LDS (two work-groups per
  // CU overlap each other's barriers and epilogues); the slab is written between two
  // barriers and the next one is already in flight in registers during the MFMAs.
  for (int kt = 0; kt < nk; ++kt) {
    const int buf = NBUF == 2 ? (kt & 1) : 0;
    if constexpr (NBUF == 1) {
      if (kt > 0) __syncthreads();
      store_lds(0);
      __syncthreads();
    }
    if (kt + 1 < nk) load_global((kt + 1) * BK);
    const bf16_t *as = As + buf * BM * PITCH + a_frag;
    const bf16_t *bs = Bs + buf * BN * PITCH + b_frag;
    // register double-buffered fragments: reads of step kk+1 go out right after the
    // first MFMA of step kk
    bf16x8 af[2][MI], bfr[2][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i) af[0][i] = *reinterpret_cast<const bf16x8 *>(as + i * 32 * PITCH);
#pragma unroll
    for (int j = 0; j < NI; ++j) bfr[0][j] = *reinterpret_cast<const bf16x8 *>(bs + j * 32 * PITCH);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int cur = kk & 1, nxt = cur ^ 1;
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[cur][j], af[cur][i], acc[i][j], 0, 0, 0);   // operands swapped: the block is C^T
          if (i == 0 && j == 0) {
            __builtin_amdgcn_sched_barrier(0);
            if (kk + 1 < BK / 16) {
#pragma unroll
              for (int i2 = 0; i2 < MI; ++i2)
                af[nxt][i2] = *reinterpret_cast<const bf16x8 *>(as + i2 * 32 * PITCH + (kk + 1) * 16);
#pragma unroll
              for (int j2 = 0; j2 < NI; ++j2)
                bfr[nxt][j2] = *reinterpret_cast<const bf16x8 *>(bs + j2 * 32 * PITCH + (kk + 1) * 16);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NBUF == 2) {
      if (kt + 1 < nk) store_lds(buf ^ 1);
      __syncthreads();
    }
  }

  const int me = m0 + wm * TM, ne = n0 + wn * TN;
  unsigned char *stg = smem + NBUF * (BM + BN) * PITCH * sizeof(bf16_t) + wave * kEpiStageBytes;
  if (me + TM <= g.M && ne + TN <= g.N) epilogue_wave<EPI, false, MI, NI>(g, acc, me, ne, lane, stg);
  else epilogue_wave<EPI, true, MI, NI>(g, acc, me, ne, lane, stg);
}

#include "gemm_pp.inc"

// ------------------------------------------------------------------ fp32 path
template <int EPI>
__device__ __forceinline__ void epilogue_store_f32(const GemmArgs &g, int m, int n, float v) {
  const size_t o = static_cast<size_t>(m) * g.ldo + n;
  float *out = static_cast<float *>(g.out);
  if constexpr (EPI == EPI_BIAS_QSCALE_ACT) {
    out[o] = (v + g.bias[n]) * (n < g.qcols ? g.qscale : 1.0f);
  } else if constexpr (EPI == EPI_BIAS_ACT || EPI == EPI_BIAS_F32) {
    out[o] = v + g.bias[n];
  } else if constexpr (EPI == EPI_BIAS_GELU_ACT) {
    out[o] = gelu_erf(v + g.bias[n]);
  } else if constexpr (EPI == EPI_BIAS_RESADD_F32) {
    out[o] = out[o] + (v + g.bias[n]);
  } else if constexpr (EPI == EPI_BIAS_ACT_GELU2) {
    out[o] = v + g.bias[n];
    static_cast<float *>(g.out2)[o] = gelu_erf(v + g.bias[n]);
  } else if constexpr (EPI == EPI_BIAS_RES_F32) {
    out[o] = static_cast<const float *>(g.aux)[o] + (v + g.bias[n]);
  } else {
    out[o] = v + g.tab[static_cast<size_t>(m % g.tab_rows) * g.N + n];
  }
}

// v_mfma_f32_32x32x2_f32 (fp32 products and sums, twice the rate of the vector pipe), operands straight from global
// memory: a lane holds row l % 32 and four consecutive k of a step of eight, so step s covers k = 8 s + 4 (l / 32) +
// 0..3 and its matrix instruction j multiplies the j-th of them, the same k on both sides.  These products are small
// and wait for memory, not for arithmetic: KS = 4 gives the four waves of a work-group the same 32 x 32 outputs and a
// quarter of the k steps each (their sums meet in LDS, added in wave order), KS = 1 gives every wave 32 x 32 outputs
// of its own once there are enough of them.  Steps are fetched AHEAD of their use.  The tiny workload's products
// (512 x 128 x 512 the longest) take 4-5 us each; the LDS-tiled vector kernel before took 22 to 70.
// VEC4: every row starts on 16 bytes.
// LN: A is the stream, normalised here (KS = 4, VEC4, K <= kLnK: a wave's part of its 32 rows stays in registers between
// the statistics and the products).  Every column tile of the output repeats that, but a LayerNorm launch of its own takes 3 us on the tiny
// workload, whatever there is to do, and this adds one: 512 x 384 x 128 and its LayerNorm 8.6 -> 6.5 us, the tiny forward 99 -> 90.
// Which products: gemm_f32_normalises().
constexpr int kLnK = 256;
template <int EPI, int KS, bool VEC4, bool LN = false>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmArgs g) {
  constexpr int AHEAD = 4;
  static_assert(!LN || (KS == 4 && VEC4), "rows in registers");
  __shared__ float part[KS == 4 ? 3 * 16 * 64 : 1];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int m0 = KS == 4 ? blockIdx.x * 32 : blockIdx.x * 64 + (wave >> 1) * 32;
  const int n0 = KS == 4 ? blockIdx.y * 32 : blockIdx.y * 64 + (wave & 1) * 32;
  size_t arow = min(m0 + l32, g.M - 1);
  if constexpr (LN) {
    if (g.a_map) arow = static_cast<size_t>(arow / g.a_out) * g.a_in + g.a_map[arow % g.a_out];
  }
  const float *a = static_cast<const float *>(g.A) + arow * g.K;
  const float *w = static_cast<const float *>(g.W) + static_cast<size_t>(min(n0 + l32, g.N - 1)) * g.K;
  const int steps = (g.K + 7) / 8, per = KS == 4 ? (steps + 3) / 4 : steps;
  const int s0 = KS == 4 ? wave * per : 0, s1 = min(steps, s0 + per);
  auto fetch = [&](const float *p, int s) {
    const int k = 8 * s + 4 * hi;
    if constexpr (VEC4) {
      return k < g.K && s < s1 ? *reinterpret_cast<const float4 *>(p + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
      const bool in = s < s1;
      return make_float4(in && k < g.K ? p[k] : 0.f, in && k + 1 < g.K ? p[k + 1] : 0.f, in && k + 2 < g.K ? p[k + 2] : 0.f,
                         in && k + 3 < g.K ? p[k + 3] : 0.f);
    }
  };
  f32x16 acc = {};
  auto multiply = [&](const float4 &x, const float4 &y) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(y.x, x.x, acc, 0, 0, 0);      // operands swapped: the block is C^T
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(y.y, x.y, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(y.z, x.z, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(y.w, x.w, acc, 0, 0, 0);
  };
  if constexpr (LN) {
    constexpr int MOST = kLnK / 8 / 4;         // steps of a wave
    __shared__ float box[2][4][32];
    float4 ra[MOST], rw[MOST], ga[MOST], be[MOST];
    auto in_row = [&](int i) { return s0 + i < s1 && 8 * (s0 + i) + 4 * hi < g.K; };
#pragma unroll
    for (int i = 0; i < MOST; ++i) ra[i] = fetch(a, s0 + i);
#pragma unroll
    for (int i = 0; i < MOST; ++i) {
      ga[i] = fetch(g.ln_g, s0 + i);
      be[i] = fetch(g.ln_b, s0 + i);
      rw[i] = fetch(w, s0 + i);
    }
    auto row_total = [&](float s, float (*b)[32]) {      // over the two lanes and the four waves that hold the row
      s += __shfl_xor(s, 32);
      if (hi == 0) b[wave][l32] = s;
      __syncthreads();
      return (b[0][l32] + b[1][l32]) + (b[2][l32] + b[3][l32]);
    };
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MOST; ++i) s += (ra[i].x + ra[i].y) + (ra[i].z + ra[i].w);
    const float mean = row_total(s, box[0]) / static_cast<float>(g.K);
    s = 0.f;
#pragma unroll
    for (int i = 0; i < MOST; ++i)
      if (in_row(i)) {
        const float x = ra[i].x - mean, y = ra[i].y - mean, z = ra[i].z - mean, u = ra[i].w - mean;
        s += (x * x + y * y) + (z * z + u * u);
      }
    const float rstd = rsqrtf(row_total(s, box[1]) / static_cast<float>(g.K) + 1e-5f);
#pragma unroll
    for (int i = 0; i < MOST; ++i) {           // gain, bias and weights past the row are zero
      const float4 v = ra[i];
      multiply(make_float4((v.x - mean) * rstd * ga[i].x + be[i].x, (v.y - mean) * rstd * ga[i].y + be[i].y,
                           (v.z - mean) * rstd * ga[i].z + be[i].z, (v.w - mean) * rstd * ga[i].w + be[i].w), rw[i]);
    }
  } else {
    float4 ra[AHEAD], rw[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      ra[i] = fetch(a, s0 + i);
      rw[i] = fetch(w, s0 + i);
    }
    for (int s = s0; s < s1; s += AHEAD) {
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {          // steps past s1 multiply zeros
        const float4 x = ra[i], y = rw[i];
        ra[i] = fetch(a, s + AHEAD + i);
        rw[i] = fetch(w, s + AHEAD + i);
        multiply(x, y);
      }
    }
  }
  const int m = m0 + l32;
  auto store = [&](int q, const float (&v)[4]) {      // registers 4 q .. 4 q + 3: columns 8 q + 4 hi + 0..3 of row l % 32
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + 8 * q + 4 * hi + j;
      if (m < g.M && n < g.N) epilogue_store_f32<EPI>(g, m, n, v[j]);
    }
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float v[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
      store(q, v);
    }
  } else {
    // every wave finishes one column quad: the others' sums of it come through LDS, wave w's part of quad q at ((w - (w > q)) * 4 + j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q != wave)
#pragma unroll
        for (int j = 0; j < 4; ++j) part[(((wave - (wave > q ? 1 : 0)) * 4 + q) * 4 + j) * 64 + lane] = acc[4 * q + j];
    __syncthreads();
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      float own = 0.f;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (q == wave) own = acc[4 * q + j];
      float s = 0.f;
#pragma unroll
      for (int o = 0; o < 4; ++o) s += o == wave ? own : part[(((o - (o > wave ? 1 : 0)) * 4 + wave) * 4 + j) * 64 + lane];
      v[j] = s;
    }
    store(wave, v);
  }
}

// ------------------------------------------------------------------ launchers
template <int BM, int BN, int BK, int WM, int WN, int NBUF, int MINW>
struct TileCfg {
  static constexpr int kBM = BM, kBN = BN, kBK = BK, kWM = WM, kWN = WN, kNBUF = NBUF, kMINW = MINW;
  static constexpr int kThreads = WM * WN * 64;
  // operand slabs + the epilogue's staging area of every wave
  static constexpr size_t kLds = static_cast<size_t>(NBUF) * (BM + BN) * (BK + 8) * sizeof(bf16_t) + WM * WN * kEpiStageBytes;
};

template <class TC, int EPI>
static hipError_t set_attr() {
  return hipFuncSetAttribute(
      reinterpret_cast<const void *>(&gemm_bf16_kernel<TC::kBM, TC::kBN, TC::kBK, TC::kWM, TC::kWN, TC::kNBUF, TC::kMINW, EPI>),
      hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(TC::kLds));
}

template <class TC, int EPI>
static hipError_t launch_bf16_tc(GemmArgs g, hipStream_t st) {
  g.grid_m = (g.M + TC::kBM - 1) / TC::kBM;
  g.grid_n = (g.N + TC::kBN - 1) / TC::kBN;
  const int total = g.grid_m * g.grid_n;
  // Narrow outputs (up to four column tiles): putting the tiles that share an A panel
  // on consecutive work-groups keeps them in step, so the panel is fetched from HBM
  // once (measured -4% on the N = 512 products of c1, +7% on the N = 2048 one).
  if (g.grid_n <= 4) g.col_fast = 1;
  gemm_bf16_kernel<TC::kBM, TC::kBN, TC::kBK, TC::kWM, TC::kWN, TC::kNBUF, TC::kMINW, EPI>
      <<<dim3(total), dim3(TC::kThreads), TC::kLds, st>>>(g);
  return hipGetLastError();
}

typedef TileCfg<128, 128, 64, 2, 2, 1, 3> TileSmall;   // 64x64 per wave, 36 KB LDS, 3 WG / CU

static int g_col_fast = 0;
static int g_gemm_tile_override = -1;   // test / tuning hook: 2 = 128x128 tiles, 3 / 4 = persistent 256x256 / 128x256

template <int EPI>
static constexpr GemmEpi epi_cost() {
  if (EPI == EPI_BIAS_GELU_ACT) return kEpiGelu;
  if (EPI == EPI_BIAS_ACT_GELU2) return kEpiTwo;
  if (EPI == EPI_BIAS_F32) return kEpiF32;
  if (EPI == EPI_BIAS_RESADD_F32 || EPI == EPI_BIAS_RES_F32 || EPI == EPI_BIAS_TAB_F32) return kEpiStream;
  return kEpiAct;
}

template <int EPI>
static hipError_t launch_bf16(GemmArgs g, hipStream_t st) {
  switch (g_gemm_tile_override >= 0 ? g_gemm_tile_override : gemm_choose(g.M, g.N, g.K, epi_cost<EPI>(), g_num_cus)) {
    case kGemm256x256: return launch_bf16_pp<2, EPI>(g, st);
    case kGemm128x256: return launch_bf16_pp<1, EPI>(g, st);
    default: return launch_bf16_tc<TileSmall, EPI>(g, st);
  }
}

static bool f32_split(int M, int N) {      // four waves to a 32 x 32 tile
  return static_cast<int64_t>((M + 31) / 32) * ((N + 31) / 32) < 8LL * g_num_cus;
}

template <int EPI>
static hipError_t launch_f32(GemmArgs g, hipStream_t st) {
  // four waves to a 32 x 32 tile while that is what it takes to give every CU two work-groups' worth of waves
  const bool split = f32_split(g.M, g.N);
  const bool vec = g.K % 4 == 0 && ((reinterpret_cast<uintptr_t>(g.A) | reinterpret_cast<uintptr_t>(g.W)) & 15) == 0;
  const int e = split ? 32 : 64;
  const dim3 grid((g.M + e - 1) / e, (g.N + e - 1) / e);
  if (grid.y > 65535) return hipErrorInvalidValue;
  if (split && vec) gemm_f32_kernel<EPI, 4, true><<<grid, dim3(256), 0, st>>>(g);
  else if (split) gemm_f32_kernel<EPI, 4, false><<<grid, dim3(256), 0, st>>>(g);
  else if (vec) gemm_f32_kernel<EPI, 1, true><<<grid, dim3(256), 0, st>>>(g);
  else gemm_f32_kernel<EPI, 1, false><<<grid, dim3(256), 0, st>>>(g);
  return hipGetLastError();
}

bool gemm_takes_layernorm(int dtype, const void *A, const void *W, const float *ln_g, const float *ln_b, int M, int N, int K) {
  return dtype == RESLIM_F32 && M > 0 && N > 0 && K > 0 && K <= kLnK && K % 4 == 0 && gemm_f32_normalises(M, N, K, g_num_cus) && f32_split(M, N) && (N + 31) / 32 <= 65535 &&
         ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(W) | reinterpret_cast<uintptr_t>(ln_g) | reinterpret_cast<uintptr_t>(ln_b)) & 15) == 0;
}

hipError_t launch_layernorm_gemm(Epilogue epi, const float *x, const ResRowMap *rows, const float *ln_g, const float *ln_b, const float *W,
                                 const float *bias, float *out, int M, int N, int K, hipStream_t st) {
  if (!gemm_takes_layernorm(RESLIM_F32, x, W, ln_g, ln_b, M, N, K)) return hipErrorInvalidValue;
  GemmArgs g = {};
  g.A = x; g.W = W; g.bias = bias; g.out = out; g.ldo = N; g.tab_rows = 1; g.M = M; g.N = N; g.K = K;
  g.qscale = 1.0f;
  g.ln_g = ln_g; g.ln_b = ln_b;
  g.a_map = rows ? rows->map : nullptr; g.a_out = rows ? rows->rows_out : 1; g.a_in = rows ? rows->rows_in : 1;
  const dim3 grid((M + 31) / 32, (N + 31) / 32), blk(256);
  if (epi == EPI_BIAS_ACT) gemm_f32_kernel<EPI_BIAS_ACT, 4, true, true><<<grid, blk, 0, st>>>(g);
  else if (epi == EPI_BIAS_GELU_ACT) gemm_f32_kernel<EPI_BIAS_GELU_ACT, 4, true, true><<<grid, blk, 0, st>>>(g);
  else if (epi == EPI_BIAS_F32) gemm_f32_kernel<EPI_BIAS_F32, 4, true, true><<<grid, blk, 0, st>>>(g);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int EPI>
static hipError_t init_epi() {
  hipError_t e;
  if ((e = set_attr_pp<2, EPI>()) != hipSuccess) return e;
  if ((e = set_attr_pp<1, EPI>()) != hipSuccess) return e;
  return set_attr<TileSmall, EPI>();
}

bool gemm_pinned() { return g_gemm_tile_override >= 0; }

hipError_t gemm_init() {
  hipError_t e;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
    g_num_cus = cus;
  if ((e = init_epi<EPI_BIAS_ACT>()) != hipSuccess) return e;
  if ((e = init_epi<EPI_BIAS_GELU_ACT>()) != hipSuccess) return e;
  if ((e = init_epi<EPI_BIAS_RESADD_F32>()) != hipSuccess) return e;
  if ((e = init_epi<EPI_BIAS_TAB_F32>()) != hipSuccess) return e;
  if ((e = init_epi<EPI_BIAS_QSCALE_ACT>()) != hipSuccess) return e;
  if ((e = init_epi<EPI_BIAS_ACT_GELU2>()) != hipSuccess) return e;
  if ((e = init_epi<EPI_BIAS_RES_F32>()) != hipSuccess) return e;
  return init_epi<EPI_BIAS_F32>();
}

hipError_t launch_gemm(int dtype, Epilogue epi, const void *A, const void *W, const float *bias,
                       void *out, int ldo, const float *tab, int tab_rows, int M, int N, int K,
                       hipStream_t st, float qscale, int qcols, const void *aux, void *out2, const ResRowMap *res_map) {
  if (M <= 0 || N <= 0 || K <= 0) return hipErrorInvalidValue;
  GemmArgs g = {};
  g.A = A; g.W = W; g.bias = bias; g.out = out; g.tab = tab;
  g.ldo = ldo; g.tab_rows = tab_rows > 0 ? tab_rows : 1;
  g.M = M; g.N = N; g.K = K; g.grid_m = g.grid_n = 0; g.col_fast = g_col_fast;
  g.qscale = qscale; g.qcols = qcols; g.aux = aux; g.out2 = out2;
  if (epi == EPI_BIAS_RES_F32 && !aux) return hipErrorInvalidValue;
  g.res_map = nullptr; g.res_out = 1; g.res_in = 1;
  if (res_map) {   // bf16 path only: the fp32 kernel reads the skip input at the output's own index
    if (epi != EPI_BIAS_RES_F32 || dtype != RESLIM_BF16 || !res_map->map || res_map->rows_out < 1) return hipErrorInvalidValue;
    g.res_map = res_map->map; g.res_out = res_map->rows_out; g.res_in = res_map->rows_in;
  }
  if (epi == EPI_BIAS_ACT_GELU2 && !out2) return hipErrorInvalidValue;
  if (dtype == RESLIM_BF16) {
    if (K % 64 != 0) return hipErrorInvalidValue;   // slabs are 64 deep; create() enforces D % 64 == 0
    if (ldo % 8 != 0 || N % 8 != 0) return hipErrorInvalidValue;  // epilogues move 16 bytes of a row at once
    if (epi == EPI_BIAS_QSCALE_ACT && qcols % 32 != 0) return hipErrorInvalidValue;   // one factor per block of 32 columns
    switch (epi) {
      case EPI_BIAS_ACT: return launch_bf16<EPI_BIAS_ACT>(g, st);
      case EPI_BIAS_GELU_ACT: return launch_bf16<EPI_BIAS_GELU_ACT>(g, st);
      case EPI_BIAS_RESADD_F32: return launch_bf16<EPI_BIAS_RESADD_F32>(g, st);
      case EPI_BIAS_TAB_F32: return launch_bf16<EPI_BIAS_TAB_F32>(g, st);
      case EPI_BIAS_QSCALE_ACT: return launch_bf16<EPI_BIAS_QSCALE_ACT>(g, st);
      case EPI_BIAS_ACT_GELU2: return launch_bf16<EPI_BIAS_ACT_GELU2>(g, st);
      case EPI_BIAS_RES_F32: return launch_bf16<EPI_BIAS_RES_F32>(g, st);
      default: return launch_bf16<EPI_BIAS_F32>(g, st);
    }
  }
  switch (epi) {
    case EPI_BIAS_ACT: return launch_f32<EPI_BIAS_ACT>(g, st);
    case EPI_BIAS_GELU_ACT: return launch_f32<EPI_BIAS_GELU_ACT>(g, st);
    case EPI_BIAS_RESADD_F32: return launch_f32<EPI_BIAS_RESADD_F32>(g, st);
    case EPI_BIAS_TAB_F32: return launch_f32<EPI_BIAS_TAB_F32>(g, st);
    case EPI_BIAS_QSCALE_ACT: return launch_f32<EPI_BIAS_QSCALE_ACT>(g, st);
    case EPI_BIAS_ACT_GELU2: return launch_f32<EPI_BIAS_ACT_GELU2>(g, st);
    case EPI_BIAS_RES_F32: return launch_f32<EPI_BIAS_RES_F32>(g, st);
    default: return launch_f32<EPI_BIAS_F32>(g, st);
  }
}

}  // namespace reslim

// tuning hook for the benchmark (not part of the method; selects the bf16 GEMM kernel: -1 heuristic, 2 = 128x128 tiles,
// 3 = persistent 256x256, 4 = persistent 128x256; +100 = columns-fastest bands)
extern "C" void reslim_debug_set_gemm_tile(int choice) {
  reslim::g_col_fast = choice >= 100 ? 1 : 0;   // 100 + c: choice c with columns-fastest bands
  reslim::g_gemm_tile_override = choice >= 100 ? choice - 100 : choice;
}
