// Gradient of tile-local multi-head self-attention (ORBIT-2 Sec. 4.2; the paper's
// headline numbers are training runs, Sec. 5).  The paper gives no formula of its
// own; this is the chain rule through  P = softmax(Q K^T / sqrt(dh)),  O = P V  for
// the tokens of one tile:
//     dV = P^T dO,   dP = dO V^T,   dS = P o (dP - delta),   delta_i = dO_i . O_i,
//     dQ = dS K / sqrt(dh),   dK = dS^T Q / sqrt(dh).
// P is never stored by the forward: it is recomputed here from Q, K and the
// log-sum-exp of every query that the forward returns.
//
// bf16 path = two launches (four at head dimension 256), no atomics, deterministic:
//   1. KV=0   query-stationary:  dQ.  It has every query's dO in registers and makes delta_i, written together with -lse_i*sqrt(dh) as
//             16-byte records (see below).  At head dimension 256 a launch before it does, attn_bwd_prep: two passes over memory
//             (80,704 tokens of 16 heads of 64 features, when it was a launch there: 93 us, 19,584 of 4: 6.6 us);
//   2. KV=1   key-stationary:    dK and dV (at head dimension 256 in two launches, half of the head's features each).
// Each head dimension has one kernel template for both: attn_bwd_woven at 64, attn_bwd_wide at 128, attn_bwd at 256.
// As in the forward kernel a work unit is 128 "stationary" tokens of one (sample, tile, head), 32
// per wave, kept in registers as MFMA B operands; the other side of the tile is streamed through
// LDS in blocks of 32 tokens (global -> LDS directly).  Every product is computed
// transposed so that a lane owns one stationary token and the streamed index runs
// over the accumulator registers:
//     Sx  = Y1 X1^T      (stream x stationary)   Y1 = K | Q,   X1 = Q | K
//     dPx = Y2 X2^T                              Y2 = V | dO,  X2 = dO | V
//     P = exp2(c Sx - lse2),  dS = P o (dPx - delta)          (fp32, in registers)
//     acc1^T += Y1^T dS      (-> dQ^T | dK^T)     the accumulators of Sx/dPx are,
//     acc2^T += Y2^T P       (-> dV^T, KV only)   rounded to bf16, directly B operands
// Y1/Y2 are read from LDS twice: as 16-byte row fragments (A operand of the first
// pair of products) and through the transposing read ds_read_b64_tr_b16 (A operand
// of the second pair).  One XOR swizzle of the 16-byte chunks of a row keeps both
// access patterns free of bank conflicts.
//
// lse and delta belong to the QUERY.  Query-stationary: they are per-lane constants
// and enter as the initial value of the accumulator chains.  Key-stationary: the query
// is the register index, so they enter through one more MFMA step instead of 2 x 16
// per-register subtractions: the streamed block carries, per query, a 16-byte record
// with the value split into three bf16 summands (exact to 2^-24), multiplied by an
// all-ones B operand (lane half 0 feeds Sx, lane half 1 feeds dPx).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "attention_common.h"
#include "attention_plan.h"
#include "gelu.h"

namespace reslim {

struct AttnBwdArgs {
  const bf16_t *qkv;     // [B, n_h, 3, heads, dh]
  const bf16_t *dout;    // [B, n_h, D]
  u32x4 *aux;            // [2][B * heads * n_h] records: 0: -lse*sqrt(dh), 1: -delta; three bf16 summands + padding
  const bf16_t *out;     // [B, n_h, D]          (head dimensions 64 and 128: the query-stationary launch makes the records)
  const float *lse;      // [B, heads, n_h]
  float lse_f;           // factor of lse in record 0
  bf16_t *dqkv;          // [B, n_h, 3, heads, dh]
  const tile_desc *tiles;
  int T, heads, D, QB, total;
  int first;             // head dimension 64: slot of the launch's first work-group
  int per;               // head dimension 128: blocks of 128 tokens of one sample and head, 0: `total` counts slots of QB a tile
  int part;              // which 1/NSPLIT of the head's features this launch accumulates and writes
  int64_t n_h;
  int64_t aux_stride;    // records per array
  float c;               // MFMA output -> base-2 logit: log2(e) / sqrt(dh)   (1 when q is pre-scaled)
  float scq, sck;        // output factors of dQ and dK: 1 / sqrt(dh) both; with pre-scaled q dK takes ln 2
};

__device__ __forceinline__ u32x4 split3_bf16(float x) {
  const bf16_t h = f32_to_bf16(x);
  const float r1 = x - bf16_to_f32(h);
  const bf16_t m = f32_to_bf16(r1);
  const float r2 = r1 - bf16_to_f32(m);
  const bf16_t l = f32_to_bf16(r2);
  u32x4 o = {static_cast<uint32_t>(h) | (static_cast<uint32_t>(m) << 16), static_cast<uint32_t>(l), 0u, 0u};
  return o;
}
__device__ __forceinline__ float join3_bf16(uint32_t w0, uint32_t w1) {
  return bf16_to_f32(static_cast<bf16_t>(w0 & 0xffffu)) + bf16_to_f32(static_cast<bf16_t>(w0 >> 16)) +
         bf16_to_f32(static_cast<bf16_t>(w1 & 0xffffu));
}

// head dimension 256: delta[b, head, tok] = sum over the head's features of dO * O; one thread per 8 features
__global__ __launch_bounds__(256) void attn_bwd_prep_bf16_kernel(const bf16_t *out, const bf16_t *dout, const float *lse,
                                                                 u32x4 *aux, int64_t n_vec, int64_t n_h, int heads,
                                                                 int D, float lse_factor, int64_t aux_stride) {
  constexpr int LPH = 256 / 8;  // lanes per head
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const bool live = idx < n_vec;
  const int64_t i = live ? idx : 0;
  const u32x4 a = *reinterpret_cast<const u32x4 *>(out + i * 8);
  const u32x4 b = *reinterpret_cast<const u32x4 *>(dout + i * 8);
  float acc = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    acc = fmaf(__uint_as_float(a[e] << 16), __uint_as_float(b[e] << 16), acc);
    acc = fmaf(__uint_as_float(a[e] & 0xffff0000u), __uint_as_float(b[e] & 0xffff0000u), acc);
  }
#pragma unroll
  for (int w = 1; w < LPH; w <<= 1) acc += __shfl_xor(acc, w);
  const int vpr = D / 8;
  const int c8 = static_cast<int>(i % vpr);
  if (live && c8 % LPH == 0) {
    const int64_t row = i / vpr;
    const int head = c8 / LPH;
    const int64_t rec = (row / n_h * heads + head) * n_h + row % n_h;
    aux[rec] = split3_bf16(-lse[rec] * lse_factor);
    aux[aux_stride + rec] = split3_bf16(-acc);
  }
}

// Head dimension 256.
// KV: keys stationary, dK and dV; else queries, dQ.
// QS: q in qkv already carries the factor log2(e)/sqrt(dh) (as the fused QKV epilogue of the
// block leaves it): the MFMA output is the base-2 logit itself.
// NSPLIT: a launch accumulates only 1 / NSPLIT of the head's output features (a.part says which)
// and recomputes the scores for each part: the accumulators of dK and dV do not fit the
// register file next to the stationary fragments.
constexpr int kBwd256Stages = 3;
constexpr int bwd256_lds_bytes(bool kv) { return kBwd256Stages * (2 * 32 * 512 + (kv ? 2 * 32 * 16 : 0)); }

template <bool KV, bool QS, int NSPLIT>
__global__ __launch_bounds__(256, 1) void attn_bwd_bf16_kernel(AttnBwdArgs a) {
  constexpr int DH = 256;
  constexpr int BS = 32;                  // streamed tokens of a block
  constexpr int NST = kBwd256Stages;      // ring of stages
  constexpr int NW = 4;
  constexpr int BX = 32 * NW;             // stationary tokens per unit: 32 per wave
  constexpr int ROWB = DH * 2;
  constexpr int CPR = DH / 8;
  constexpr int RPB = 64 / CPR;
  constexpr int TILE_B = BS * ROWB;
  constexpr int AUXB = KV ? 2 * BS * 16 : 0;
  constexpr int AUXL = AUXB / 1024;       // wave-loads of the record block
  constexpr int STAGE = 2 * TILE_B + AUXB;
  constexpr int LPW = TILE_B / 1024 / NW;
  constexpr int NKS = DH / 16, NDT = DH / 32 / NSPLIT;   // NDT: 32-feature blocks of the accumulators
  static_assert(TILE_B % (1024 * NW) == 0 && AUXB % 1024 == 0 && NST * STAGE == bwd256_lds_bytes(KV), "LDS plan");
  extern __shared__ __align__(1024) unsigned char smem[];   // NST * STAGE bytes

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int ldq = 3 * a.D;
  const int ldx2 = KV ? ldq : a.D, ldy2 = KV ? a.D : ldq;
  const int G = gridDim.x;
  // chunk swizzle of a row, good for both the 16-byte row fragments (16 lanes, 16 rows, one
  // chunk column) and the transposing reads (32 lanes, 4 consecutive rows x 4 chunks)
  auto swz = [](int r) {
    return ((r & 3) << 2) | ((r >> 2) & 3);
  };

  // A unit = 128 stationary tokens of one (sample, tile, head); everything is uniform over the
  // work-group and kept as element offsets so that a descriptor costs few scalar registers.
  struct Unit {
    int n_t, r0, nsb;
    int64_t q_off;      // first element of the tile's q rows of this head in qkv / d_qkv
    int64_t o_off;      // ... of its rows in d_out
    int64_t aux_off;    // ... of its records in record array 0
  };
  auto decode = [&](int vb, Unit &u) -> int {      // first non-empty unit at or after vb (stride G), or >= total
    while (vb < a.total) {
      const int logical = xcd_remap_attn(vb, a.total);
      const int xb = logical % a.QB;
      int rest = logical / a.QB;
      const int head = rest % a.heads;
      rest /= a.heads;
      const int tile = rest % a.T;
      const int b = rest / a.T;
      const int n_t = a.tiles[tile].n_tok;
      if (xb * BX < n_t) {
        const int64_t row0 = static_cast<int64_t>(b) * a.n_h + a.tiles[tile].tok_off;
        u.n_t = n_t;
        u.r0 = xb * BX;
        u.nsb = (n_t + BS - 1) / BS;
        u.q_off = row0 * ldq + head * DH;
        u.o_off = row0 * a.D + head * DH;
        u.aux_off = (static_cast<int64_t>(b) * a.heads + head) * a.n_h + a.tiles[tile].tok_off;
        return vb;
      }
      vb += G;
    }
    return vb;
  };
  auto x1_of = [&](const Unit &u) { return a.qkv + u.q_off + (KV ? a.D : 0); };
  auto x2_of = [&](const Unit &u) { return KV ? a.qkv + u.q_off + 2 * a.D : a.dout + u.o_off; };
  auto y1_of = [&](const Unit &u) { return a.qkv + u.q_off + (KV ? 0 : a.D); };
  auto y2_of = [&](const Unit &u) { return KV ? a.dout + u.o_off : a.qkv + u.q_off + 2 * a.D; };
  Unit cur, nxt;
  int vb = decode(blockIdx.x, cur);
  if (vb >= a.total) return;
  // the loads run NST - 1 blocks ahead of the arithmetic, across unit boundaries: a second
  // cursor walks the same sequence of (unit, block)
  Unit iu = cur;
  int ivb = vb, iblk = 0;
  vb = decode(vb + G, nxt);
  bool has_next = vb < a.total;

  // ---- load side: lane -> (row of the block, 16-byte chunk), per-lane byte offsets
  int ld_row[LPW], off1[LPW], off2[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    ld_row[i] = (wave + NW * i) * RPB + lane / CPR;
    const int ch = ((lane % CPR) ^ swz(ld_row[i])) * 16;
    off1[i] = ld_row[i] * ldq * 2 + ch;
    off2[i] = ld_row[i] * ldy2 * 2 + ch;
  }
  const int aux_L = wave * 64 + lane;                 // record slot of this lane in the block (KV only)
  const int aux_arr = aux_L / BS, aux_row = aux_L % BS;
  auto issue = [&](const Unit &u, int s0, int buf) {
    unsigned char *sb = smem + buf * STAGE;
    const unsigned char *g1 = reinterpret_cast<const unsigned char *>(y1_of(u) + static_cast<size_t>(s0) * ldq);
    const unsigned char *g2 = reinterpret_cast<const unsigned char *>(y2_of(u) + static_cast<size_t>(s0) * ldy2);
    const int lim = u.n_t - 1 - s0;       // last valid row of this block
    if (lim >= BS - 1) {                   // whole block inside the tile (uniform)
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        attn_dl_load16(reinterpret_cast<const bf16_t *>(g1 + static_cast<uint32_t>(off1[i])), sb + (wave + NW * i) * 1024);
        attn_dl_load16(reinterpret_cast<const bf16_t *>(g2 + static_cast<uint32_t>(off2[i])),
                       sb + TILE_B + (wave + NW * i) * 1024);
      }
    } else {                               // rows past the tile end re-read its last row (finite; masked later)
#pragma unroll
      for (int i = 0; i < LPW; ++i) {
        const int back = max(ld_row[i] - lim, 0);
        attn_dl_load16(reinterpret_cast<const bf16_t *>(g1 + static_cast<uint32_t>(off1[i] - back * ldq * 2)),
                       sb + (wave + NW * i) * 1024);
        attn_dl_load16(reinterpret_cast<const bf16_t *>(g2 + static_cast<uint32_t>(off2[i] - back * ldy2 * 2)),
                       sb + TILE_B + (wave + NW * i) * 1024);
      }
    }
    if constexpr (KV) {
      if (wave < AUXL) {
        const int row = s0 + min(aux_row, lim);
        attn_dl_load16(reinterpret_cast<const bf16_t *>(a.aux + u.aux_off + aux_arr * a.aux_stride + row),
                       sb + 2 * TILE_B + wave * 1024);
      }
    }
  };
  bf16x8 x1f[NKS], x2f[NKS];
  f32x16 sinit, dpinit;
  auto load_x = [&](const Unit &u) {
    const int xrow = min(u.r0 + wave * 32 + l32, u.n_t - 1);
    const bf16_t *p1 = x1_of(u) + static_cast<size_t>(xrow) * ldq + hi * 8;
    const bf16_t *p2 = x2_of(u) + static_cast<size_t>(xrow) * ldx2 + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      x1f[ks] = *reinterpret_cast<const bf16x8 *>(p1 + ks * 16);
      x2f[ks] = *reinterpret_cast<const bf16x8 *>(p2 + ks * 16);
    }
    float si = 0.f, di = 0.f;
    if constexpr (!KV) {
      const u32x2 r0 = *reinterpret_cast<const u32x2 *>(a.aux + u.aux_off + xrow);
      const u32x2 r1 = *reinterpret_cast<const u32x2 *>(a.aux + u.aux_off + a.aux_stride + xrow);
      si = join3_bf16(r0[0], r0[1]);
      di = join3_bf16(r1[0], r1[1]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) { sinit[r] = si; dpinit[r] = di; }
  };

  // ---- read side
  // Row fragment: A-operand row l32 carries streamed token key_perm(l32) of its 32-token group.
  // Transposed fragment: this lane points at token row 8*hi + 4*e + (lane%16)/4 of a 16-token
  // step and at the 4 features 32*d + 16*((lane/16)&1) + 4*(lane%4) .. +3.
  const int yr = key_perm(l32);
  const int y_row = yr * ROWB, y_swz = swz(yr);
  const int L16 = lane & 15;
  int t_addr[2][NDT];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int vr = 8 * hi + 4 * e + (L16 >> 2);
#pragma unroll
    for (int d = 0; d < NDT; ++d) {
      const int o = 32 * (d + a.part * NDT) + 16 * ((lane >> 4) & 1) + 4 * (L16 & 3);
      t_addr[e][d] = vr * ROWB + (((o >> 3) ^ swz(vr)) << 4) + ((o >> 2) & 1) * 8;
    }
  }
  const int aux_addr = 2 * TILE_B + hi * BS * 16 + yr * 16;

  // all-ones B operands of the record step: lane half 0 -> Sx, lane half 1 -> dPx
  bf16x8 ones_s, ones_d;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ones_s[e] = static_cast<__bf16>(e < 3 && hi == 0 ? 1.0f : 0.0f);
    ones_d[e] = static_cast<__bf16>(e < 3 && hi == 1 ? 1.0f : 0.0f);
  }

  f32x16 acc1[NDT], acc2[KV ? NDT : 1];
  auto reset = [&]() {
#pragma unroll
    for (int d = 0; d < NDT; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc1[d][r] = 0.f;
#pragma unroll
    for (int d = 0; d < (KV ? NDT : 1); ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc2[d][r] = 0.f;
  };
  reset();
  load_x(cur);
  // issue the next block of the load cursor into stage `buf`; false when the sequence has ended
  auto issue_next = [&](int buf) -> bool {
    if (ivb >= a.total) return false;
    issue(iu, iblk * BS, buf);
    if (++iblk == iu.nsb) {
      ivb = decode(ivb + G, iu);
      iblk = 0;
    }
    return true;
  };
  constexpr int NLD = 2 * LPW;            // direct loads of one block per wave (+1 in the waves that fetch records)
  int ahead = 0;                          // blocks in flight beyond the one about to be computed
  issue_next(0);
#pragma unroll
  for (int i = 1; i < NST - 1; ++i) ahead += issue_next(i) ? 1 : 0;

  int sb = 0, buf = 0;
  for (;;) {
    // block `sb` of `cur` must have landed; younger blocks may stay in flight.  Loads complete in
    // issue order, so "at most `ahead` blocks' worth outstanding" is enough.
    if (ahead == 0) {
      __builtin_amdgcn_s_waitcnt(0x0F70);
    } else if (KV && wave < AUXL) {
      __builtin_amdgcn_s_waitcnt(0x0F70 | ((NLD + 1) & 15) | (((NLD + 1) >> 4) << 14));
    } else {
      __builtin_amdgcn_s_waitcnt(0x0F70 | (NLD & 15) | ((NLD >> 4) << 14));
    }
    // a bare barrier: __syncthreads() would add a fence that waits for ALL vector-memory operations,
    // the younger prefetches included.  Every wave has waited for its own direct-to-LDS loads of
    // this block above, and LDS reads of the stage being refilled finished before its readers arrived.
    __builtin_amdgcn_s_barrier();           // everybody's part of the block is in LDS; the oldest stage is free
    const bool last = sb + 1 == cur.nsb;
    const bool active = cur.r0 + wave * 32 < cur.n_t;
    {
      int ibuf = buf + NST - 1;
      if (ibuf >= NST) ibuf -= NST;
      if (!issue_next(ibuf) && ahead > 0) --ahead;      // one computed, one issued: `ahead` unchanged
    }
    const unsigned char *st = smem + buf * STAGE;
    const int s0 = sb * BS;

    // The work on a block, in three phases.
    auto scores = [&](f32x16 &s, f32x16 &dp) {                      // matrix pipe
      // the fragment reads run PF steps ahead of the MFMAs that use them, in a ring
      // of PF + 1 register sets, and a scheduling barrier per step keeps that order (left to
      // itself the compiler either waits for every read right before its MFMA or hoists all
      // reads of the group to its top: 64+ registers of fragments next to the accumulators)
      constexpr int PF = 2;
      bf16x8 f1[PF + 1], f2[PF + 1];
      auto fetch = [&](int ks) {
        const unsigned char *rp = st + y_row + (((2 * ks + hi) ^ y_swz) << 4);
        f1[ks % (PF + 1)] = *reinterpret_cast<const bf16x8 *>(rp);
        f2[ks % (PF + 1)] = *reinterpret_cast<const bf16x8 *>(rp + TILE_B);
      };
#pragma unroll
      for (int ks = 0; ks < PF; ++ks) fetch(ks);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        if (ks + PF < NKS) fetch(ks + PF);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[ks % (PF + 1)], x1f[ks], ks == 0 ? sinit : s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[ks % (PF + 1)], x2f[ks], ks == 0 ? dpinit : dp, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (KV) {
        const bf16x8 fa = *reinterpret_cast<const bf16x8 *>(st + aux_addr);
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, ones_s, s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa, ones_d, dp, 0, 0, 0);
      }
    };
    auto mask = [&](f32x16 &s) {              // ragged end: streamed tokens past the tile end get probability 0
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = s0 + 16 * (r / 8) + 8 * hi + (r % 8);
        if (row >= cur.n_t) s[r] = -INFINITY;
      }
    };
    auto probs = [&](f32x16 &s, f32x16 &dp) {                       // vector pipe: s <- P, dp <- dS
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] = __builtin_amdgcn_exp2f(QS ? s[r] : s[r] * a.c);
        dp[r] *= s[r];
      }
    };
    auto products = [&](const f32x16 &s, const f32x16 &dp) {        // matrix pipe
      auto step = [&](auto h2_c) {
        constexpr int h2 = decltype(h2_c)::value;
        constexpr int ROFF = h2 * 16 * ROWB;
        bf16x8 pf, dsf;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          dsf[e] = static_cast<__bf16>(dp[8 * h2 + e]);
          if constexpr (KV) pf[e] = static_cast<__bf16>(s[8 * h2 + e]);
        }
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        auto tr_frag = [&](int off) {
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(st + off));
          return lo;
        };
#pragma unroll
        for (int d = 0; d < NDT; ++d) {
          {
            const s16x8 both = __builtin_shufflevector(tr_frag(ROFF + t_addr[0][d]), tr_frag(ROFF + t_addr[1][d]), 0, 1, 2, 3, 4, 5, 6, 7);
            acc1[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), dsf, acc1[d], 0, 0, 0);
          }
          if constexpr (KV) {
            const s16x8 both = __builtin_shufflevector(tr_frag(ROFF + TILE_B + t_addr[0][d]), tr_frag(ROFF + TILE_B + t_addr[1][d]), 0, 1, 2, 3, 4, 5, 6, 7);
            acc2[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf, acc2[d], 0, 0, 0);
          }
        }
      };
      step(std::integral_constant<int, 0>{});
      step(std::integral_constant<int, 1>{});
    };
    // The next unit's stationary fragments are fetched at ONE place, after the last scores that use the current ones.
    f32x16 sA, dA;
    if (active) scores(sA, dA);
    if (last && has_next) load_x(nxt);
    if (active) {
      if (s0 + BS > cur.n_t) mask(sA);
      probs(sA, dA);
      products(sA, dA);
    }
    if (++buf == NST) buf = 0;
    if (!last) { ++sb; continue; }

    // ---- end of a unit: scale, round and store this lane's row of each gradient
    const int xrow = cur.r0 + wave * 32 + l32;
    if (active && xrow < cur.n_t) {
      bf16_t *p1 = a.dqkv + cur.q_off + (KV ? a.D : 0) + static_cast<size_t>(xrow) * ldq + hi * 4 + a.part * NDT * 32;
      bf16_t *p2 = a.dqkv + cur.q_off + 2 * a.D + static_cast<size_t>(xrow) * ldq + hi * 4 + a.part * NDT * 32;
      const float sc1 = KV ? a.sck : a.scq;
#pragma unroll
      for (int d = 0; d < NDT; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          // registers 4*r4 .. 4*r4+3 hold features 32d + 8*r4 + 4*hi + (0..3) of this lane's token
          bf16x4 tmp;
#pragma unroll
          for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(acc1[d][4 * r4 + e] * sc1);
          *reinterpret_cast<u32x2 *>(p1 + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
          if constexpr (KV) {
#pragma unroll
            for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(acc2[d][4 * r4 + e]);
            *reinterpret_cast<u32x2 *>(p2 + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
          }
        }
    }
    if (!has_next) break;
    // Everything in flight (the next unit's stationary fragments, the result stores, the
    // prefetched blocks) is waited for here, once per unit: with register loads possibly
    // pending across the loop edge the compiler would otherwise wait for ALL vector-memory
    // operations, the prefetch included, before the first fragment use of every block.
    __builtin_amdgcn_s_waitcnt(0x0F70);
    cur = nxt;
    vb = decode(vb + G, nxt);
    has_next = vb < a.total;
    sb = 0;
    reset();
  }
}

// ------------------------------------------------------------------ head dimension 64: two groups of streamed tokens in flight
// A phase of a wave is 32 streamed tokens: the products of the group before (acc += Y^T dS, Y^T P), with the exponentials of this group between
// their matrix instructions, then the scores of the group after, with the rest of this group's dS and P between theirs.  So
// neither the vector work nor the LDS reads are in the matrix instructions' way: row fragments are read a phase ahead, each as soon as the one
// in its place has been used, column fragments half a phase ahead.  The order is pinned as in the forward kernel with two query groups.
// Seven or eight blocks lie in LDS, one barrier a phase: block i + 2 has landed, block i - 2 is free.  Two work-groups of four waves per
// compute unit (206 and 238 registers); they start unit after unit, not persistent, so uneven tiles even out.
// Every sum has the order of the kernel above: the same bits.  That one had scores, exponentials and products one after the other, two or three
// waves a SIMD: 80,704 tokens of 16 heads in tiles of 1128 to 1323, dQ 749 us and dK, dV 1149 there, 737 and 967 here; 2000 tokens, 16 sets of keys
// 45.4 and 57.8, 36.4 and 43.7; 30 tokens, 1024 sets 9.7 and 10.0, 8.4 and 8.3.  What bounds it: matrix pipe 45 and 51 % of the cycles, vector unit 47 and
// 42 %, at 1.85 GHz; the loads are 15 % of the time (eight waves that share them were slower still: 814 and 1057 us), the LDS reads 7 %.
template <bool KV, bool QS>
__global__ __launch_bounds__(256, 2) void attn_bwd_woven_bf16_kernel(AttnBwdArgs a) {
  constexpr int DH = 64, ROWB = DH * 2, TILE = 32 * ROWB, REC = KV ? 2 * 32 * 16 : 0, STAGE = 2 * TILE + REC, NST = KV ? 7 : 8, NKS = DH / 16;
  constexpr int LOADS = KV ? 3 : 2;                    // direct loads of a wave per block
  __shared__ __align__(1024) unsigned char smem[NST * STAGE];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int logical = a.first + xcd_remap_attn(blockIdx.x, gridDim.x);
  const int xb = logical % a.QB;
  int rest = logical / a.QB;
  const int head = rest % a.heads;
  rest /= a.heads;
  const int tile = rest % a.T, b = rest / a.T;
  const int n_t = a.tiles[tile].n_tok, x0 = xb * 128 + wave * 32;
  if (xb * 128 >= n_t) return;                         // uniform
  const int64_t row0 = static_cast<int64_t>(b) * a.n_h + a.tiles[tile].tok_off;
  const int64_t rec0 = (static_cast<int64_t>(b) * a.heads + head) * a.n_h + a.tiles[tile].tok_off;
  const int ldq = 3 * a.D, ldx2 = KV ? ldq : a.D, ldy2 = KV ? a.D : ldq;
  const bf16_t *const q = a.qkv + row0 * ldq + head * DH, *const dout = a.dout + row0 * a.D + head * DH;
  const bool active = x0 < n_t;
  const int n = (n_t + 31) / 32;                       // blocks of streamed tokens

  // ---- load side.  The buffers cover exactly the rows of a block that exist: the rest of it, and blocks past the last one, are zeros without
  // an access.  A wave loads eight rows of either operand and a quarter of the records.
  auto swz = [](int r) { return (((r >> 1) & 1) << 2) | (((r >> 2) & 1) << 1) | ((r >> 3) & 1); };
  const int l_row = wave * 8 + lane / 8, l_chunk = ((lane % 8) ^ swz(l_row)) * 16;
  const int off1 = l_row * ldq * 2 + l_chunk, off2 = l_row * ldy2 * 2 + l_chunk, off3 = (wave & 1) * 256 + lane * 4;
  const bf16_t *y1 = q + (KV ? 0 : a.D), *y2 = KV ? dout : q + 2 * a.D;
  const u32x4 *rec = a.aux + rec0 + (wave >> 1) * a.aux_stride;
  int rows_left = n_t;
  unsigned l_stage = 0;
  auto after = [](unsigned stage) { return stage == (NST - 1) * STAGE ? 0u : stage + STAGE; };
  auto buffer = [](const void *p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000); };
  auto to_lds = [&](__amdgpu_buffer_rsrc_t r, unsigned at, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(smem + at), 16, off, 0, 0, 0);
  };
  auto load_rows = [&]() {
    to_lds(buffer(y1, max((min(rows_left, 32) - 1) * ldq * 2 + ROWB, 0)), l_stage + wave * 1024, off1);
    y1 += static_cast<size_t>(32) * ldq;
  };
  auto load_rest = [&]() {
    to_lds(buffer(y2, max((min(rows_left, 32) - 1) * ldy2 * 2 + ROWB, 0)), l_stage + TILE + wave * 1024, off2);
    y2 += static_cast<size_t>(32) * ldy2;
    if constexpr (KV) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer(rec, max(min(rows_left, 32) * 16, 0)),
                                               (__attribute__((address_space(3))) void *)(smem + l_stage + 2 * TILE + wave * 256), 4, off3, 0, 0, 0);
      rec += 32;
    }
    rows_left -= 32;
    l_stage = after(l_stage);
  };
  // all but the youngest `blocks` of this wave's loads are done, then everybody's
  auto landed = [&](auto blocks) {
    constexpr int N = LOADS * decltype(blocks)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4 << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  typedef std::integral_constant<int, NST - 4> First;
  typedef std::integral_constant<int, NST - 5> Next;

  // ---- stationary side
  bf16x8 x1f[NKS], x2f[NKS];
  f32x16 sinit, dpinit;
  if (active) {
    const int xrow = min(x0 + l32, n_t - 1);
    const bf16_t *p1 = q + (KV ? a.D : 0) + static_cast<size_t>(xrow) * ldq + hi * 8;
    const bf16_t *p2 = (KV ? q + 2 * a.D : dout) + static_cast<size_t>(xrow) * ldx2 + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      x1f[ks] = *reinterpret_cast<const bf16x8 *>(p1 + ks * 16);
      x2f[ks] = *reinterpret_cast<const bf16x8 *>(p2 + ks * 16);
    }
    float si = 0.f, di = 0.f;
    if constexpr (!KV) {
      // delta of the lane's query: its upstream gradient is here, so only the output is read.  Chunks of eight features, then pairs of
      // chunks, in the order of attn_bwd_prep; a lane has the chunks of its half.  The records are for the key-stationary launch.
      const bf16_t *po = a.out + (row0 + xrow) * a.D + head * DH + hi * 8;
      float part[NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const u32x4 o = *reinterpret_cast<const u32x4 *>(po + ks * 16), g = __builtin_bit_cast(u32x4, x2f[ks]);
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc = fmaf(__uint_as_float(o[e] << 16), __uint_as_float(g[e] << 16), acc);
          acc = fmaf(__uint_as_float(o[e] & 0xffff0000u), __uint_as_float(g[e] & 0xffff0000u), acc);
        }
        unsigned lo, up;
        lane_pair_exchange(__builtin_bit_cast(unsigned, acc), lo, up);
        part[ks] = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, up);
      }
      const float delta = (part[0] + part[1]) + (part[2] + part[3]);
      const u32x4 r0 = split3_bf16(-a.lse[rec0 + xrow] * a.lse_f), r1 = split3_bf16(-delta);
      if (x0 + l32 < n_t) {
        if (hi == 0) a.aux[rec0 + xrow] = r0;
        else a.aux[a.aux_stride + rec0 + xrow] = r1;
      }
      si = join3_bf16(r0[0], r0[1]);
      di = join3_bf16(r1[0], r1[1]);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) { sinit[r] = si; dpinit[r] = di; }
  }
  // Blocks that do not exist are not waited for: what is read of them (a block ahead) is not used.  16,384 sets of keys of 33 tokens, both launches: 360 us with
  // all of the ring loaded first, 351 now; of 16 tokens 232 and 217; 4096 of 1 token 44.7 and 41.8.
  for (int i = 0; i < NST - 2 && i < n; ++i) {
    load_rows();
    load_rest();
  }
  if (n < NST - 2) __builtin_amdgcn_s_waitcnt(0x0F70);   // the counts below are of a full ring
  landed(First{});                       // blocks 0 and 1
  if (!active) {                         // loads and barriers only
    for (int i = 0; i < n; ++i) {
      landed(Next{});
      load_rows();
      load_rest();
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // no load into LDS outlives its work-group
    return;
  }

  // ---- read side: rows (a lane's token key_perm(l32), 16-byte chunks) and, through the transposing read, columns
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)smem));
  auto lds = [](unsigned at) { return *reinterpret_cast<__attribute__((address_space(3))) bf16x8 *>(at); };
  const int yr = key_perm(l32);
  const unsigned r_base = lds0 + yr * ROWB + ((hi ^ swz(yr)) << 4), rec_base = lds0 + 2 * TILE + hi * 512 + yr * 16;
  const int vr = 8 * hi + ((lane & 15) >> 2), vo = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const unsigned t_base = lds0 + vr * ROWB + (((vo >> 3) ^ swz(vr)) << 4) + ((vo >> 2) & 1) * 8;
  bf16x8 f1[NKS], f2[NKS], fr;
  unsigned r_stage = 0, t_stage = 0;
  auto read_row1 = [&](auto ks_c) __attribute__((always_inline)) { f1[decltype(ks_c)::value] = lds((r_base + r_stage) ^ (decltype(ks_c)::value * 32)); };
  auto read_row2 = [&](auto ks_c) __attribute__((always_inline)) { f2[decltype(ks_c)::value] = lds(((r_base + r_stage) ^ (decltype(ks_c)::value * 32)) + TILE); };
  auto read_record = [&]() __attribute__((always_inline)) {
    if constexpr (KV) fr = lds(rec_base + r_stage);
    r_stage = after(r_stage);
  };
  auto rows_are_there = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) asm volatile("" : "+v"(f1[ks]), "+v"(f2[ks]));
    if constexpr (KV) asm volatile("" : "+v"(fr));
  };
  // columns of 16 streamed tokens: Y1's and, keys stationary, Y2's; [block of 32 features][rows + 0..3 and + 4..7].  Issued in one statement and
  // waited for in another (see attention_common.h)
  struct Columns { uint64_t y1[2][2], y2[2][2]; };
  Columns c0, c1;
  auto issue_columns = [&](Columns &c, auto h_c) __attribute__((always_inline)) {
    constexpr int OFF = decltype(h_c)::value * 16 * ROWB;
    const unsigned at0 = t_base + t_stage, at1 = (at0 + 512) ^ 32;
    if constexpr (KV) {
      asm volatile(
          "ds_read_b64_tr_b16 %0, %8 offset:%12\n\t"
          "ds_read_b64_tr_b16 %1, %9 offset:%12\n\t"
          "ds_read_b64_tr_b16 %2, %8 offset:%13\n\t"
          "ds_read_b64_tr_b16 %3, %9 offset:%13\n\t"
          "ds_read_b64_tr_b16 %4, %10 offset:%12\n\t"
          "ds_read_b64_tr_b16 %5, %11 offset:%12\n\t"
          "ds_read_b64_tr_b16 %6, %10 offset:%13\n\t"
          "ds_read_b64_tr_b16 %7, %11 offset:%13"
          : "=&v"(c.y1[0][0]), "=&v"(c.y1[0][1]), "=&v"(c.y2[0][0]), "=&v"(c.y2[0][1]),
            "=&v"(c.y1[1][0]), "=&v"(c.y1[1][1]), "=&v"(c.y2[1][0]), "=&v"(c.y2[1][1])
          : "v"(at0), "v"(at1), "v"(at0 ^ 64u), "v"(at1 ^ 64u), "n"(OFF), "n"(OFF + TILE));
    } else {
      asm volatile(
          "ds_read_b64_tr_b16 %0, %4 offset:%8\n\t"
          "ds_read_b64_tr_b16 %1, %5 offset:%8\n\t"
          "ds_read_b64_tr_b16 %2, %6 offset:%8\n\t"
          "ds_read_b64_tr_b16 %3, %7 offset:%8"
          : "=&v"(c.y1[0][0]), "=&v"(c.y1[0][1]), "=&v"(c.y1[1][0]), "=&v"(c.y1[1][1])
          : "v"(at0), "v"(at1), "v"(at0 ^ 64u), "v"(at1 ^ 64u), "n"(OFF));
    }
  };
  auto wait_columns = [&](Columns &c) __attribute__((always_inline)) {
    if constexpr (KV) {
      asm volatile("s_waitcnt lgkmcnt(0)"
                   : "+v"(c.y1[0][0]), "+v"(c.y1[0][1]), "+v"(c.y2[0][0]), "+v"(c.y2[0][1]),
                     "+v"(c.y1[1][0]), "+v"(c.y1[1][1]), "+v"(c.y2[1][0]), "+v"(c.y2[1][1]));
    } else {
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(c.y1[0][0]), "+v"(c.y1[0][1]), "+v"(c.y1[1][0]), "+v"(c.y1[1][1]));
    }
  };
  bf16x8 ones_s, ones_d;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ones_s[e] = static_cast<__bf16>(e < 3 && hi == 0 ? 1.0f : 0.0f);
    ones_d[e] = static_cast<__bf16>(e < 3 && hi == 1 ? 1.0f : 0.0f);
  }

  f32x16 acc1[2], acc2[KV ? 2 : 1], s[2], dp[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      acc1[d][r] = 0.f;
      if constexpr (KV) acc2[d][r] = 0.f;
    }
  u32x4 pk_p[2], pk_d[2];                // P and dS of the group before, bf16 pairs
  auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
  auto score = [&](auto p_c, auto ks_c) __attribute__((always_inline)) {
    constexpr int p = decltype(p_c)::value, ks = decltype(ks_c)::value;
    if constexpr (ks == NKS) {
      s[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, ones_s, s[p], 0, 0, 0);
    } else if constexpr (ks == 0) {
      if constexpr (!KV) asm volatile("" : "+v"(sinit));
      s[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[0], x1f[0], sinit, 0, 0, 0);
      if constexpr (!KV) asm volatile("" : "+v"(s[p]), "+v"(sinit));
    } else {
      s[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[ks], x1f[ks], s[p], 0, 0, 0);
    }
  };
  auto dscore = [&](auto p_c, auto ks_c) __attribute__((always_inline)) {
    constexpr int p = decltype(p_c)::value, ks = decltype(ks_c)::value;
    if constexpr (ks == NKS) {
      dp[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, ones_d, dp[p], 0, 0, 0);
    } else if constexpr (ks == 0) {
      if constexpr (!KV) asm volatile("" : "+v"(dpinit));
      dp[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[0], x2f[0], dpinit, 0, 0, 0);
      if constexpr (!KV) asm volatile("" : "+v"(dp[p]), "+v"(dpinit));
    } else {
      dp[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[ks], x2f[ks], dp[p], 0, 0, 0);
    }
  };
  typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
  auto product1 = [&](const Columns &c, auto h_c, auto d_c) __attribute__((always_inline)) {
    constexpr int h2 = decltype(h_c)::value, d = decltype(d_c)::value;
    const u64x2 y = {c.y1[d][0], c.y1[d][1]};
    acc1[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, y), __builtin_bit_cast(bf16x8, pk_d[h2]), acc1[d], 0, 0, 0);
  };
  auto product2 = [&](const Columns &c, auto h_c, auto d_c) __attribute__((always_inline)) {
    constexpr int h2 = decltype(h_c)::value, d = decltype(d_c)::value;
    if constexpr (KV) {
      const u64x2 y = {c.y2[d][0], c.y2[d][1]};
      acc2[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, y), __builtin_bit_cast(bf16x8, pk_p[h2]), acc2[d], 0, 0, 0);
    }
  };
  auto exps = [&](auto p_c, auto r_c, auto n_c) __attribute__((always_inline)) {      // P of values r .. r + n - 1
    constexpr int p = decltype(p_c)::value, r = decltype(r_c)::value, N = decltype(n_c)::value;
#pragma unroll
    for (int k = 0; k < N; k += 2) {
      float e0 = __builtin_amdgcn_exp2f(QS ? s[p][r + k] : s[p][r + k] * a.c), e1 = __builtin_amdgcn_exp2f(QS ? s[p][r + k + 1] : s[p][r + k + 1] * a.c);
      asm volatile("" : "+v"(e0), "+v"(e1));
      s[p][r + k] = e0; s[p][r + k + 1] = e1;
    }
  };
  auto finish = [&](auto p_c, auto k_c) __attribute__((always_inline)) {              // dS and the bf16 pair k
    constexpr int p = decltype(p_c)::value, k = decltype(k_c)::value;
    uint32_t d = pack2(dp[p][2 * k] * s[p][2 * k], dp[p][2 * k + 1] * s[p][2 * k + 1]);
    asm volatile("" : "+v"(d));
    pk_d[k / 4][k % 4] = d;
    if constexpr (KV) {
      uint32_t v = pack2(s[p][2 * k], s[p][2 * k + 1]);
      asm volatile("" : "+v"(v));
      pk_p[k / 4][k % 4] = v;
    }
  };
  auto mask = [&](auto p_c, int blk) __attribute__((always_inline)) {                 // streamed tokens past the tile end get probability 0
    constexpr int p = decltype(p_c)::value;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (blk * 32 + 16 * (r / 8) + 8 * hi + (r % 8) >= n_t) s[p][r] = -INFINITY;
  };
#define RESLIM_I(n) std::integral_constant<int, n>{}
  // Phase of block blk, whose scores are in s[P] and dp[P]: first the products of the block before (where pr) with the exponentials between them,
  // then the scores of the block after (past the last one: of zeros, not used) with the rest of dS between them.
  auto phase = [&](auto p_c, auto pr, int blk) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value;
    constexpr bool PR = decltype(pr)::value;
    std::integral_constant<int, 1 - P> o_c;
    landed(Next{});                      // block blk + 2; everybody has left block blk - 2
    if (__builtin_expect(blk * 32 + 32 > n_t, 0)) mask(p_c, blk);
    if constexpr (PR) {
      wait_columns(c0);
      if constexpr (KV) issue_columns(c1, RESLIM_I(1));
      else wait_columns(c1);
      if constexpr (KV) t_stage = after(t_stage);
    }
    if constexpr (KV) {
      fence();
      if constexpr (PR) product1(c0, RESLIM_I(0), RESLIM_I(0));
      fence();
      load_rows();
      exps(p_c, RESLIM_I(0), RESLIM_I(2));
      fence();
      if constexpr (PR) product2(c0, RESLIM_I(0), RESLIM_I(0));
      fence();
      load_rest();
      exps(p_c, RESLIM_I(2), RESLIM_I(2));
      fence();
      if constexpr (PR) product1(c0, RESLIM_I(0), RESLIM_I(1));
      fence();
      exps(p_c, RESLIM_I(4), RESLIM_I(2));
      fence();
      if constexpr (PR) product2(c0, RESLIM_I(0), RESLIM_I(1));
      fence();
      exps(p_c, RESLIM_I(6), RESLIM_I(2));
      if constexpr (PR) wait_columns(c1);
      fence();
      if constexpr (PR) product1(c1, RESLIM_I(1), RESLIM_I(0));
      fence();
      exps(p_c, RESLIM_I(8), RESLIM_I(2));
      fence();
      if constexpr (PR) product2(c1, RESLIM_I(1), RESLIM_I(0));
      fence();
      exps(p_c, RESLIM_I(10), RESLIM_I(2));
      fence();
      if constexpr (PR) product1(c1, RESLIM_I(1), RESLIM_I(1));
      fence();
      exps(p_c, RESLIM_I(12), RESLIM_I(2));
      fence();
      if constexpr (PR) product2(c1, RESLIM_I(1), RESLIM_I(1));
      fence();
      exps(p_c, RESLIM_I(14), RESLIM_I(2));
      fence();
    } else {
      if constexpr (PR) product1(c0, RESLIM_I(0), RESLIM_I(0));
      fence();
      load_rows();
      exps(p_c, RESLIM_I(0), RESLIM_I(4));
      fence();
      if constexpr (PR) product1(c0, RESLIM_I(0), RESLIM_I(1));
      fence();
      load_rest();
      exps(p_c, RESLIM_I(4), RESLIM_I(4));
      fence();
      if constexpr (PR) product1(c1, RESLIM_I(1), RESLIM_I(0));
      fence();
      exps(p_c, RESLIM_I(8), RESLIM_I(4));
      fence();
      if constexpr (PR) product1(c1, RESLIM_I(1), RESLIM_I(1));
      fence();
      exps(p_c, RESLIM_I(12), RESLIM_I(4));
      fence();
    }
    rows_are_there();
    fence();
    score(o_c, RESLIM_I(0));
    fence();
    read_row1(RESLIM_I(0));
    finish(p_c, RESLIM_I(0));
    fence();
    dscore(o_c, RESLIM_I(0));
    fence();
    read_row2(RESLIM_I(0));
    finish(p_c, RESLIM_I(1));
    fence();
    score(o_c, RESLIM_I(1));
    fence();
    read_row1(RESLIM_I(1));
    finish(p_c, RESLIM_I(2));
    fence();
    dscore(o_c, RESLIM_I(1));
    fence();
    read_row2(RESLIM_I(1));
    finish(p_c, RESLIM_I(3));
    fence();
    score(o_c, RESLIM_I(2));
    fence();
    read_row1(RESLIM_I(2));
    finish(p_c, RESLIM_I(4));
    fence();
    dscore(o_c, RESLIM_I(2));
    fence();
    read_row2(RESLIM_I(2));
    issue_columns(c0, RESLIM_I(0));
    if constexpr (!KV) {
      issue_columns(c1, RESLIM_I(1));
      t_stage = after(t_stage);
    }
    finish(p_c, RESLIM_I(5));
    fence();
    score(o_c, RESLIM_I(3));
    fence();
    read_row1(RESLIM_I(3));
    finish(p_c, RESLIM_I(6));
    fence();
    dscore(o_c, RESLIM_I(3));
    fence();
    read_row2(RESLIM_I(3));
    finish(p_c, RESLIM_I(7));
    fence();
    if constexpr (KV) {
      score(o_c, RESLIM_I(NKS));
      dscore(o_c, RESLIM_I(NKS));
      fence();
    }
    read_record();
    fence();
  };
  typedef std::integral_constant<int, 0> Even;
  typedef std::integral_constant<int, 1> Odd;
  typedef std::true_type Yes;
  typedef std::false_type No;

  auto read_rows = [&]() __attribute__((always_inline)) {
    read_row1(RESLIM_I(0)); read_row2(RESLIM_I(0));
    read_row1(RESLIM_I(1)); read_row2(RESLIM_I(1));
    read_row1(RESLIM_I(2)); read_row2(RESLIM_I(2));
    read_row1(RESLIM_I(3)); read_row2(RESLIM_I(3));
    read_record();
  };
  read_rows();
  rows_are_there();
  score(Even{}, RESLIM_I(0)); dscore(Even{}, RESLIM_I(0));
  score(Even{}, RESLIM_I(1)); dscore(Even{}, RESLIM_I(1));
  score(Even{}, RESLIM_I(2)); dscore(Even{}, RESLIM_I(2));
  score(Even{}, RESLIM_I(3)); dscore(Even{}, RESLIM_I(3));
  if constexpr (KV) { score(Even{}, RESLIM_I(NKS)); dscore(Even{}, RESLIM_I(NKS)); }
  read_rows();
  phase(Even{}, No{}, 0);
  int i = 1;
#pragma unroll 1
  for (; i + 1 < n; i += 2) {
    phase(Odd{}, Yes{}, i);
    phase(Even{}, Yes{}, i + 1);
  }
  if (i < n) phase(Odd{}, Yes{}, i);
  wait_columns(c0);
  if constexpr (KV) {
    issue_columns(c1, RESLIM_I(1));
    wait_columns(c1);
  } else {
    wait_columns(c1);
  }
  product1(c0, RESLIM_I(0), RESLIM_I(0)); product2(c0, RESLIM_I(0), RESLIM_I(0));
  product1(c0, RESLIM_I(0), RESLIM_I(1)); product2(c0, RESLIM_I(0), RESLIM_I(1));
  product1(c1, RESLIM_I(1), RESLIM_I(0)); product2(c1, RESLIM_I(1), RESLIM_I(0));
  product1(c1, RESLIM_I(1), RESLIM_I(1)); product2(c1, RESLIM_I(1), RESLIM_I(1));
#undef RESLIM_I
  __builtin_amdgcn_s_waitcnt(0x0F70);    // no load into LDS outlives its work-group

  // ---- scale, round and store this lane's row of each gradient
  const int xrow = x0 + l32;
  if (xrow >= n_t) return;
  bf16_t *p1 = a.dqkv + row0 * ldq + head * DH + (KV ? a.D : 0) + static_cast<size_t>(xrow) * ldq + hi * 4, *p2 = p1 + a.D;
  const float sc1 = KV ? a.sck : a.scq;
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      // registers 4*r4 .. 4*r4+3 hold features 32d + 8*r4 + 4*hi + (0..3) of this lane's token
      bf16x4 tmp;
#pragma unroll
      for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(acc1[d][4 * r4 + e] * sc1);
      *reinterpret_cast<u32x2 *>(p1 + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
      if constexpr (KV) {
#pragma unroll
        for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(acc2[d][4 * r4 + e]);
        *reinterpret_cast<u32x2 *>(p2 + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
      }
    }
}

// ------------------------------------------------------------------ head dimension 128: the same weave, one wave a SIMD
// The phases of attn_bwd_woven, with twice the products for the same exponentials: 24 matrix instructions a phase query-stationary, 34
// key-stationary.  The accumulators, the stationary rows and a phase's fragments take 398 and 419 registers, so one wave a SIMD and nothing else to fill its
// gaps: the second half of a block's rows is read during the products, and columns and rows lie in accumulator registers, which the matrix
// instructions read as well and vector code does not need.  One work-group to a compute unit walks its units; the loads run six blocks ahead across
// units, and the next unit's stationary rows arrive during a unit's last products.  Every sum has the order of the kernel for head dimension 256: the same bits.
// 19,840 tokens of 24 heads in tiles of 1128 to 1323: 1564 us with two groups one after the other and three stages of 64 tokens, 1201 us here;
// 37,536 of 32 in tiles to 2448: 6.69 and 5.05 ms; 2000 tokens, 8 sets of keys 150 and 115 us; 30 tokens, 1024 sets 53 and 48.
// What bounds it: the matrix pipe is busy 39 and 44 % of the cycles, at 1.94 GHz; a wave issues 47 % of the time, waits for LDS, loads and the barrier 22 and 21 %, and for
// a busy unit the rest.
// Exponentials and loads spread evenly over both halves of the phase measured the same.
template <int N, typename F, int... I>
__device__ __forceinline__ void each_of(const F &f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
__device__ __forceinline__ int64_t scalar64(int64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v)), up = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
  return static_cast<int64_t>(static_cast<uint64_t>(up) << 32 | lo);
}
__device__ __forceinline__ void pin2(bf16x8 &x, bf16x8 &y) { asm volatile("" : "+a"(x), "+a"(y)); }
template <int N, typename F>
__device__ __forceinline__ void each(const F &f) { each_of<N>(f, std::make_integer_sequence<int, N>{}); }

constexpr int kWideStages = 8;
constexpr int wide_lds_bytes(bool kv) { return kWideStages * (2 * 32 * 256 + (kv ? 2 * 32 * 16 : 0)); }

template <bool KV, bool QS>
__global__ __launch_bounds__(256, 1) void attn_bwd_wide_bf16_kernel(AttnBwdArgs a) {
  constexpr int DH = 128, ROWB = DH * 2, TILE = 32 * ROWB, STAGE = wide_lds_bytes(KV) / kWideStages, NST = kWideStages, NKS = DH / 16, ND = DH / 32;
  constexpr int LOADS = KV ? 5 : 4;                    // direct loads of a wave per block
  extern __shared__ __align__(1024) unsigned char smem[];   // wide_lds_bytes(KV)
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int ldq = 3 * a.D, ldx2 = KV ? ldq : a.D, ldy2 = KV ? a.D : ldq;
  const int G = gridDim.x;
  struct Unit {
    int n_t, x0, head;   // tokens of the tile; first stationary token of the work-group
    int64_t row0, rec0;  // first row of the tile, first record of its head
  };
  // Unit `vb` of the launch: of the blocks of 128 tokens that exist, over samples, heads and tiles; every wave finds the tile with a running sum
  // over the tiles, a lane each.  Where that does not pay (a.per == 0, see the launch) of the slots of as many blocks as the longest tile
  // has, empty ones skipped, stride G.
  auto decode = [&](int vb, Unit &u) __attribute__((always_inline)) -> int {         // vb, or the next slot that has a block; >= total: none
    int b = 0, tile = 0;
    while (vb < a.total) {
      const int logical = xcd_remap_attn(vb, a.total);
      if (a.per) {
        int at = logical % a.per, rest = logical / a.per;
        u.head = rest % a.heads;
        b = rest / a.heads;
        const int own = lane < a.T ? (a.tiles[lane].n_tok + 127) / 128 : 0;
        int upto = own;
#pragma unroll
        for (int w = 1; w < 64; w <<= 1) {
          const int v = __shfl_up(upto, w);
          upto += lane >= w ? v : 0;
        }
        tile = __builtin_ctzll(__ballot(upto > at));
        u.x0 = (at - __builtin_amdgcn_readlane(upto - own, tile)) * 128;
      } else {
        int rest = logical / a.QB;
        u.x0 = logical % a.QB * 128;
        u.head = rest % a.heads;
        rest /= a.heads;
        tile = rest % a.T;
        b = rest / a.T;
      }
      // the kernel writes to memory, so these come through vector loads: back to scalar registers, or the buffers' addresses are not
      u.n_t = __builtin_amdgcn_readfirstlane(a.tiles[tile].n_tok);
      const int64_t off = scalar64(a.tiles[tile].tok_off);
      u.row0 = static_cast<int64_t>(b) * a.n_h + off;
      u.rec0 = (static_cast<int64_t>(b) * a.heads + u.head) * a.n_h + off;
      if (u.x0 < u.n_t) break;
      vb += G;
    }
    return vb;
  };
  auto q_of = [&](const Unit &u) __attribute__((always_inline)) { return a.qkv + u.row0 * ldq + u.head * DH; };
  auto dout_of = [&](const Unit &u) __attribute__((always_inline)) { return a.dout + u.row0 * a.D + u.head * DH; };
  Unit cur;
  int vb = decode(blockIdx.x, cur);
  if (vb >= a.total) return;                           // uniform

  // ---- load side, ahead of the arithmetic across units.  The buffers cover exactly the rows of a block that exist: the rest of it, and
  // blocks past the last unit, are zeros without an access.  A wave loads eight rows of either operand and a quarter of the records.
  auto swz = [](int r) { return ((r & 3) << 2) | ((r >> 2) & 3); };
  int off1[2], off2[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = wave * 8 + i * 4 + lane / 16, chunk = ((lane % 16) ^ swz(row)) * 16;
    off1[i] = row * ldq * 2 + chunk;
    off2[i] = row * ldy2 * 2 + chunk;
  }
  const int off3 = (wave & 1) * 256 + lane * 4;
  // at least two, so that a unit's first and last phase are two: a second block of a short tile is of zeros, masked like any row past the end
  auto blocks_of = [](int n_t) { return max((n_t + 31) / 32, 2); };
  int lvb = vb, rows_left = 0, blocks_left = 0;
  const bf16_t *y1 = nullptr, *y2 = nullptr;
  const u32x4 *rec = nullptr;
  unsigned l_stage = 0;
  auto after = [](unsigned stage) { return stage == (NST - 1) * STAGE ? 0u : stage + STAGE; };
  auto buffer = [](const void *p, int bytes) { return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, bytes, 0x00020000); };
  auto to_lds = [&](__amdgpu_buffer_rsrc_t r, unsigned at, int off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(smem + at), 16, off, 0, 0, 0);
  };
  auto load_from = [&](const Unit &u) __attribute__((always_inline)) {
    y1 = q_of(u) + (KV ? 0 : a.D);
    y2 = KV ? dout_of(u) : q_of(u) + 2 * a.D;
    rec = a.aux + u.rec0 + (wave >> 1) * a.aux_stride;
    rows_left = u.n_t;
    blocks_left = blocks_of(u.n_t);
  };
  auto load_rows = [&]() __attribute__((always_inline)) {
    const auto r = buffer(y1, max((min(rows_left, 32) - 1) * ldq * 2 + ROWB, 0));
    to_lds(r, l_stage + wave * 2048, off1[0]);
    to_lds(r, l_stage + wave * 2048 + 1024, off1[1]);
    y1 += static_cast<size_t>(32) * ldq;
  };
  auto load_rest = [&]() __attribute__((always_inline)) {
    const auto r = buffer(y2, max((min(rows_left, 32) - 1) * ldy2 * 2 + ROWB, 0));
    to_lds(r, l_stage + TILE + wave * 2048, off2[0]);
    to_lds(r, l_stage + TILE + wave * 2048 + 1024, off2[1]);
    y2 += static_cast<size_t>(32) * ldy2;
    if constexpr (KV) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(buffer(rec, max(min(rows_left, 32) * 16, 0)),
                                               (__attribute__((address_space(3))) void *)(smem + l_stage + 2 * TILE + wave * 256), 4, off3, 0, 0, 0);
      rec += 32;
    }
    rows_left -= 32;
    --blocks_left;
    l_stage = after(l_stage);
  };
  auto next_to_load = [&]() __attribute__((always_inline)) {   // before a block's loads: the next unit, where this one has no block left
    if (blocks_left <= 0 && lvb < a.total) {
      Unit u;
      lvb = decode(lvb + G, u);
      if (lvb < a.total) load_from(u);
    }
  };
  // all but the youngest `blocks` of this wave's loads are done, then everybody's
  auto landed = [&](auto blocks) __attribute__((always_inline)) {
    constexpr int N = LOADS * decltype(blocks)::value;
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4 << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  typedef std::integral_constant<int, NST - 4> First;
  typedef std::integral_constant<int, NST - 5> Next;

  // ---- stationary side: fetch() starts the loads of a unit's, settle() needs them done
  bf16x8 x1f[NKS], x2f[NKS];
  u32x4 o_row[KV ? 1 : NKS];
  float lse_x = 0.f;
  f32x16 sinit, dpinit;
  auto fetch = [&](const Unit &u) __attribute__((always_inline)) {
    const int xrow = min(u.x0 + wave * 32 + l32, u.n_t - 1);
    const bf16_t *p1 = q_of(u) + (KV ? a.D : 0) + static_cast<size_t>(xrow) * ldq + hi * 8;
    const bf16_t *p2 = (KV ? q_of(u) + 2 * a.D : dout_of(u)) + static_cast<size_t>(xrow) * ldx2 + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      x1f[ks] = *reinterpret_cast<const bf16x8 *>(p1 + ks * 16);
      x2f[ks] = *reinterpret_cast<const bf16x8 *>(p2 + ks * 16);
    }
    if constexpr (!KV) {
      const bf16_t *po = a.out + (u.row0 + xrow) * a.D + u.head * DH + hi * 8;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) o_row[ks] = *reinterpret_cast<const u32x4 *>(po + ks * 16);
      lse_x = a.lse[u.rec0 + xrow];
    }
  };
  auto settle = [&](const Unit &u) __attribute__((always_inline)) {
    float si = 0.f, di = 0.f;
    if constexpr (!KV) {
      // delta of the lane's query: chunks of eight features, then pairs of chunks, in the order of attn_bwd_prep; a lane has the chunks
      // of its half.  The records are for the key-stationary launch.
      float part[NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const u32x4 o = o_row[ks], g = __builtin_bit_cast(u32x4, x2f[ks]);
        float acc = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          acc = fmaf(__uint_as_float(o[e] << 16), __uint_as_float(g[e] << 16), acc);
          acc = fmaf(__uint_as_float(o[e] & 0xffff0000u), __uint_as_float(g[e] & 0xffff0000u), acc);
        }
        unsigned lo, up;
        lane_pair_exchange(__builtin_bit_cast(unsigned, acc), lo, up);
        part[ks] = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, up);
      }
      const float delta = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
      const u32x4 r0 = split3_bf16(-lse_x * a.lse_f), r1 = split3_bf16(-delta);
      const int xrow = u.x0 + wave * 32 + l32;
      if (xrow < u.n_t) {
        if (hi == 0) a.aux[u.rec0 + xrow] = r0;
        else a.aux[a.aux_stride + u.rec0 + xrow] = r1;
      }
      si = join3_bf16(r0[0], r0[1]);
      di = join3_bf16(r1[0], r1[1]);
    }
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) pin2(x1f[ks], x2f[ks]);
#pragma unroll
    for (int r = 0; r < 16; ++r) { sinit[r] = si; dpinit[r] = di; }
  };

  // ---- read side: rows (a lane's token key_perm(l32), 16-byte chunks) and, through the transposing read, columns
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)smem));
  auto lds = [](unsigned at) __attribute__((always_inline)) { return *reinterpret_cast<__attribute__((address_space(3))) bf16x8 *>(at); };
  const int yr = key_perm(l32);
  const unsigned r_base = lds0 + yr * ROWB + ((hi ^ swz(yr)) << 4), rec_base = lds0 + 2 * TILE + hi * 512 + yr * 16;
  const int vr = 8 * hi + ((lane & 15) >> 2), vo = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const unsigned t_base = lds0 + vr * ROWB + (((vo >> 3) ^ swz(vr)) << 4) + ((vo >> 2) & 1) * 8;
  bf16x8 f1[NKS], f2[NKS], fr;
  unsigned r_stage = 0, t_stage = 0;
  auto read_row1 = [&](auto ks_c) __attribute__((always_inline)) { f1[decltype(ks_c)::value] = lds((r_base + r_stage) ^ (decltype(ks_c)::value * 32)); };
  auto read_row2 = [&](auto ks_c) __attribute__((always_inline)) { f2[decltype(ks_c)::value] = lds(((r_base + r_stage) ^ (decltype(ks_c)::value * 32)) + TILE); };
  auto read_record = [&]() __attribute__((always_inline)) {
    if constexpr (KV) {
      fr = lds(rec_base + r_stage);
    }
  };
  auto half_is_there = [&](auto h_c) __attribute__((always_inline)) {
    constexpr int h = decltype(h_c)::value;
#pragma unroll
    for (int ks = h * NKS / 2; ks < (h + 1) * NKS / 2; ++ks) pin2(f1[ks], f2[ks]);
  };
  // columns of 16 streamed tokens of one operand: [block of 32 features][rows + 0..3 and + 4..7].  Issued in one statement and waited for in another
  // (see attention_common.h)
  typedef uint64_t Columns[ND][2];
  Columns c1[2], c2[KV ? 2 : 1];
  auto issue_columns = [&](Columns &c, auto off_c) __attribute__((always_inline)) {
    const unsigned at0 = t_base + t_stage, at1 = (at0 + 1024) ^ 16;
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%16\n\t"
        "ds_read_b64_tr_b16 %1, %9 offset:%16\n\t"
        "ds_read_b64_tr_b16 %2, %10 offset:%16\n\t"
        "ds_read_b64_tr_b16 %3, %11 offset:%16\n\t"
        "ds_read_b64_tr_b16 %4, %12 offset:%16\n\t"
        "ds_read_b64_tr_b16 %5, %13 offset:%16\n\t"
        "ds_read_b64_tr_b16 %6, %14 offset:%16\n\t"
        "ds_read_b64_tr_b16 %7, %15 offset:%16"
        : "=&a"(c[0][0]), "=&a"(c[0][1]), "=&a"(c[1][0]), "=&a"(c[1][1]), "=&a"(c[2][0]), "=&a"(c[2][1]), "=&a"(c[3][0]), "=&a"(c[3][1])
        : "v"(at0), "v"(at1), "v"(at0 ^ 64u), "v"(at1 ^ 64u), "v"(at0 ^ 128u), "v"(at1 ^ 128u), "v"(at0 ^ 192u), "v"(at1 ^ 192u),
          "n"(decltype(off_c)::value));
  };
  auto wait_columns = [&](Columns &c) __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+a"(c[0][0]), "+a"(c[0][1]), "+a"(c[1][0]), "+a"(c[1][1]), "+a"(c[2][0]), "+a"(c[2][1]), "+a"(c[3][0]), "+a"(c[3][1]));
  };
  auto issue1 = [&](auto h_c) __attribute__((always_inline)) { issue_columns(c1[decltype(h_c)::value], std::integral_constant<int, decltype(h_c)::value * 16 * ROWB>{}); };
  auto issue2 = [&](auto h_c) __attribute__((always_inline)) {
    if constexpr (KV) issue_columns(c2[decltype(h_c)::value], std::integral_constant<int, decltype(h_c)::value * 16 * ROWB + TILE>{});
  };
  auto wait_half = [&](auto h_c) __attribute__((always_inline)) {
    wait_columns(c1[decltype(h_c)::value]);
    if constexpr (KV) wait_columns(c2[decltype(h_c)::value]);
  };
  bf16x8 ones_s, ones_d;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ones_s[e] = static_cast<__bf16>(e < 3 && hi == 0 ? 1.0f : 0.0f);
    ones_d[e] = static_cast<__bf16>(e < 3 && hi == 1 ? 1.0f : 0.0f);
  }

  asm volatile("" : "+a"(ones_s), "+a"(ones_d));

  f32x16 acc1[ND], acc2[KV ? ND : 1], s[2], dp[2];
  u32x4 pk_p[2], pk_d[2];                // P and dS of the group before, bf16 pairs
  int n_t = 0;
  auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
  auto score = [&](auto p_c, auto ks_c) __attribute__((always_inline)) {
    constexpr int p = decltype(p_c)::value, ks = decltype(ks_c)::value;
    if constexpr (ks == NKS) {
      s[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, ones_s, s[p], 0, 0, 0);
    } else if constexpr (ks == 0) {
      if constexpr (!KV) asm volatile("" : "+v"(sinit));
      s[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[0], x1f[0], sinit, 0, 0, 0);
      if constexpr (!KV) asm volatile("" : "+v"(s[p]), "+v"(sinit));
    } else {
      s[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f1[ks], x1f[ks], s[p], 0, 0, 0);
    }
  };
  auto dscore = [&](auto p_c, auto ks_c) __attribute__((always_inline)) {
    constexpr int p = decltype(p_c)::value, ks = decltype(ks_c)::value;
    if constexpr (ks == NKS) {
      dp[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr, ones_d, dp[p], 0, 0, 0);
    } else if constexpr (ks == 0) {
      if constexpr (!KV) asm volatile("" : "+v"(dpinit));
      dp[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[0], x2f[0], dpinit, 0, 0, 0);
      if constexpr (!KV) asm volatile("" : "+v"(dp[p]), "+v"(dpinit));
    } else {
      dp[p] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f2[ks], x2f[ks], dp[p], 0, 0, 0);
    }
  };
  typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
  // product j of a group: 16 streamed tokens h2, 32 features d; keys stationary dK and dV in turn
  constexpr int NP = KV ? 4 * ND : 2 * ND;
  auto product = [&](auto j_c) __attribute__((always_inline)) {
    constexpr int h2 = decltype(j_c)::value / (NP / 2), i = decltype(j_c)::value % (NP / 2), d = KV ? i / 2 : i;
    if constexpr (!KV || i % 2 == 0) {
      const u64x2 y = {c1[h2][d][0], c1[h2][d][1]};
      acc1[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, y), __builtin_bit_cast(bf16x8, pk_d[h2]), acc1[d], 0, 0, 0);
    } else {
      const u64x2 y = {c2[h2][d][0], c2[h2][d][1]};
      acc2[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, y), __builtin_bit_cast(bf16x8, pk_p[h2]), acc2[d], 0, 0, 0);
    }
  };
  auto exp_of = [&](auto p_c, auto r_c) __attribute__((always_inline)) {              // P
    constexpr int p = decltype(p_c)::value, r = decltype(r_c)::value;
    float e = __builtin_amdgcn_exp2f(QS ? s[p][r] : s[p][r] * a.c);
    asm volatile("" : "+v"(e));
    s[p][r] = e;
  };
  auto finish = [&](auto p_c, auto k_c) __attribute__((always_inline)) {              // dS and the bf16 pair k
    constexpr int p = decltype(p_c)::value, k = decltype(k_c)::value;
    uint32_t d = pack2(dp[p][2 * k] * s[p][2 * k], dp[p][2 * k + 1] * s[p][2 * k + 1]);
    asm volatile("" : "+v"(d));
    pk_d[k / 4][k % 4] = d;
    if constexpr (KV) {
      uint32_t v = pack2(s[p][2 * k], s[p][2 * k + 1]);
      asm volatile("" : "+v"(v));
      pk_p[k / 4][k % 4] = v;
    }
  };
  auto mask = [&](auto p_c, int blk) __attribute__((always_inline)) {                 // streamed tokens past the tile end get probability 0
    constexpr int p = decltype(p_c)::value;
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (blk * 32 + 16 * (r / 8) + 8 * hi + (r % 8) >= n_t) s[p][r] = -INFINITY;
  };
  typedef std::integral_constant<int, 0> Even;
  typedef std::integral_constant<int, 1> Odd;
  typedef std::true_type Yes;
  typedef std::false_type No;
  // First half of the phase of block blk, whose scores are in s[P] and dp[P]: the products of the block before (where pr) with the exponentials and the second
  // half of the rows of block blk + 1 between them.
  auto products = [&](auto p_c, auto pr, int blk) __attribute__((always_inline)) {
    constexpr bool PR = decltype(pr)::value;
    next_to_load();
    landed(Next{});                      // block blk + 2; everybody has left block blk - 2
    if (__builtin_expect(blk * 32 + 32 > n_t, 0)) mask(p_c, blk);
    if constexpr (PR) {
      wait_half(Even{});
      if constexpr (KV) {
        issue1(Odd{});
        issue2(Odd{});
        t_stage = after(t_stage);
      } else {
        wait_half(Odd{});
      }
    }
    fence();
    each<NP>([&](auto j_c) __attribute__((always_inline)) {
      constexpr int j = decltype(j_c)::value, E = 16 / NP, R = NP - 8;       // E exponentials an instruction; rows from instruction R on
      if constexpr (PR) {
        if constexpr (KV && j == NP / 2) wait_half(Odd{});
        product(j_c);
        fence();
      }
      if constexpr (j == 0) load_rows();
      if constexpr (j == 1) load_rest();
      each<E>([&](auto e_c) __attribute__((always_inline)) { exp_of(p_c, std::integral_constant<int, j * E + decltype(e_c)::value>{}); });
      if constexpr (j >= R && (j - R) % 2 == 0) read_row1(std::integral_constant<int, NKS / 2 + (j - R) / 2>{});
      if constexpr (j >= R && (j - R) % 2 == 1) read_row2(std::integral_constant<int, NKS / 2 + (j - R) / 2>{});
      fence();
    });
    read_record();
    r_stage = after(r_stage);
    fence();
  };
  // Second half: the scores of the block after (where sc) with the rest of dS (where fin) and the first half of the rows of the block after that between
  // them, and the columns of this block.
  auto scores = [&](auto p_c, auto fin, auto sc) __attribute__((always_inline)) {
    constexpr int P = decltype(p_c)::value;
    constexpr bool FIN = decltype(fin)::value, SC = decltype(sc)::value;
    std::integral_constant<int, 1 - P> o_c;
    if constexpr (SC) half_is_there(Even{});
    fence();
    each<NKS>([&](auto ks_c) __attribute__((always_inline)) {
      constexpr int ks = decltype(ks_c)::value;
      if constexpr (SC) {
        if constexpr (ks == NKS / 2) half_is_there(Odd{});
        fence();
        score(o_c, ks_c);
        fence();
        if constexpr (ks < NKS / 2) read_row1(ks_c);
      }
      if constexpr (FIN) {
        if constexpr (ks == (SC ? NKS / 2 + KV : 0)) issue1(Even{});
        finish(p_c, ks_c);
        fence();
      }
      if constexpr (SC) {
        dscore(o_c, ks_c);
        fence();
        if constexpr (ks < NKS / 2) read_row2(ks_c);
      }
      if constexpr (FIN) {
        if constexpr (ks == (SC ? NKS / 2 + 2 : 0)) {
          if constexpr (KV) {
            issue2(Even{});
          } else {
            issue1(Odd{});
            t_stage = after(t_stage);
          }
        }
        fence();
      }
    });
    if constexpr (SC && KV) {
      score(o_c, std::integral_constant<int, NKS>{});
      dscore(o_c, std::integral_constant<int, NKS>{});
    }
    fence();
  };

  load_from(cur);
  for (int i = 0; i < NST - 2; ++i) {
    next_to_load();
    load_rows();
    load_rest();
  }
  fetch(cur);
  __builtin_amdgcn_s_waitcnt(0x0F70);
  landed(First{});                       // blocks 0 and 1
  unsigned stage0 = 0;                   // of the unit's first block
  for (;;) {
    n_t = cur.n_t;
    const int n = blocks_of(n_t), x0 = cur.x0 + wave * 32;
    if (x0 < n_t) {
      settle(cur);
      r_stage = t_stage = stage0;
      each<NKS>([&](auto ks_c) __attribute__((always_inline)) { read_row1(ks_c); read_row2(ks_c); });
      read_record();
      r_stage = after(r_stage);
#pragma unroll
      for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc1[d][r] = 0.f;
          if constexpr (KV) acc2[d][r] = 0.f;
        }
      scores(Odd{}, No{}, Yes{});
      // Phases 0 .. n - 1.  Scores change between s[0], dp[0] and s[1], dp[1]; the last phase, which has none to compute, is always one with s[1].
      products(Even{}, No{}, 0);
      scores(Even{}, Yes{}, Yes{});
      int i = 1;
#pragma unroll 1
      for (; i + 2 < n; i += 2) {
        products(Odd{}, Yes{}, i);
        scores(Odd{}, Yes{}, Yes{});
        products(Even{}, Yes{}, i + 1);
        scores(Even{}, Yes{}, Yes{});
      }
      if (i + 1 < n) {
        products(Odd{}, Yes{}, i);
        scores(Odd{}, Yes{}, Yes{});
        s[1] = s[0];
        dp[1] = dp[0];
      }
      products(Odd{}, Yes{}, n - 1);
      scores(Odd{}, Yes{}, No{});
      if constexpr (KV) {
        issue1(Odd{});
        issue2(Odd{});
      }
      wait_half(Even{});
      wait_half(Odd{});
    } else {                             // loads and barriers only
      for (int i = 0; i < n; ++i) {
        next_to_load();
        landed(Next{});
        load_rows();
        load_rest();
      }
    }
    Unit nxt;
    vb = decode(vb + G, nxt);
    const bool more = vb < a.total;
    if (more) fetch(nxt);                // while the last products are computed and this lane's row of each gradient is scaled, rounded and stored
    const int xrow = x0 + l32;
    if (x0 < n_t) each<NP>([&](auto j_c) __attribute__((always_inline)) { product(j_c); });
    if (xrow < n_t) {
      bf16_t *p1 = a.dqkv + cur.row0 * ldq + cur.head * DH + (KV ? a.D : 0) + static_cast<size_t>(xrow) * ldq + hi * 4, *p2 = p1 + a.D;
      const float sc1 = KV ? a.sck : a.scq;
#pragma unroll
      for (int d = 0; d < ND; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          // registers 4*r4 .. 4*r4+3 hold features 32d + 8*r4 + 4*hi + (0..3) of this lane's token
          bf16x4 tmp;
#pragma unroll
          for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(acc1[d][4 * r4 + e] * sc1);
          *reinterpret_cast<u32x2 *>(p1 + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
          if constexpr (KV) {
#pragma unroll
            for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(acc2[d][4 * r4 + e]);
            *reinterpret_cast<u32x2 *>(p2 + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
          }
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // the next unit's rows are there; after the last unit no load into LDS outlives its work-group
    if (!more) return;
    stage0 = (stage0 / STAGE + n) % NST * STAGE;
    cur = nxt;
  }
}

// ------------------------------------------------------------------ fp32 path
__global__ __launch_bounds__(256) void attn_bwd_delta_f32_kernel(const float *out, const float *dout, float *delta,
                                                                 int64_t n, int64_t n_h, int heads, int dh) {
  // one thread per (sample, token, head)
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= n) return;
  const int head = static_cast<int>(idx % heads);
  const int64_t row = idx / heads;
  const float *o = out + (row * heads + head) * dh;
  const float *d_o = dout + (row * heads + head) * dh;
  float acc = 0.f;
  for (int d = 0; d < dh; ++d) acc = fmaf(o[d], d_o[d], acc);
  delta[(row / n_h * heads + head) * n_h + row % n_h] = acc;
}

// KV = false: one work-group per query token, gradient of q.  KV = true: one per key token, gradients of k and v.
template <bool KV>
__global__ __launch_bounds__(128) void attn_bwd_f32_kernel(const float *qkv, const float *dout, const float *lse,
                                                           const float *delta, float *dqkv, const tile_desc *tiles,
                                                           const int32_t *tile_of_tok, int64_t n_h, int heads, int D,
                                                           int dh, int max_n_tok) {
  extern __shared__ float sm[];
  float *wds = sm;                      // [max_n_tok] dS towards every token of the other side
  float *wp = sm + max_n_tok;           // [max_n_tok] P (KV only)
  float *x1 = sm + 2 * max_n_tok;       // [dh] this token's q (or k)
  float *x2 = x1 + dh;                  // [dh] this token's dO (or v)
  const int64_t tok = blockIdx.x;
  const int head = blockIdx.y, b = blockIdx.z;
  const int tile = tile_of_tok[tok];
  const int n_t = tiles[tile].n_tok;
  const int64_t tok_off = tiles[tile].tok_off;
  const int ld = 3 * D;
  const size_t row_b = static_cast<size_t>(b) * n_h;
  const float *qb = qkv + (row_b + tok_off) * ld + head * dh;             // q of the tile's first token
  const float *dob = dout + (row_b + tok_off) * D + head * dh;
  const float *stat = lse + (static_cast<size_t>(b) * heads + head) * n_h;
  const float *dstat = delta + (static_cast<size_t>(b) * heads + head) * n_h;
  const float *mine = qkv + (row_b + tok) * ld + head * dh;
  const int t = threadIdx.x;
  for (int d = t; d < dh; d += 128) {
    x1[d] = KV ? mine[D + d] : mine[d];
    x2[d] = KV ? mine[2 * D + d] : dout[(row_b + tok) * D + head * dh + d];
  }
  __syncthreads();
  const float scale = rsqrtf(static_cast<float>(dh));
  for (int j = t; j < n_t; j += 128) {
    // KV: j is a query, this token the key; else j is a key, this token the query
    const float *y1 = qb + static_cast<size_t>(j) * ld + (KV ? 0 : D);
    const float *y2 = KV ? dob + static_cast<size_t>(j) * D : qb + static_cast<size_t>(j) * ld + 2 * D;
    float s = 0.f, dp = 0.f;
    for (int d = 0; d < dh; ++d) {
      s = fmaf(x1[d], y1[d], s);
      dp = fmaf(x2[d], y2[d], dp);
    }
    const int64_t qi = KV ? tok_off + j : tok;
    const float p = expf(s * scale - stat[qi]);
    wds[j] = p * (dp - dstat[qi]);
    if (KV) wp[j] = p;
  }
  __syncthreads();
  float *go = dqkv + (row_b + tok) * ld + head * dh;
  for (int d = t; d < dh; d += 128) {
    float a1 = 0.f, a2 = 0.f;
    for (int j = 0; j < n_t; ++j) {
      a1 = fmaf(wds[j], qb[static_cast<size_t>(j) * ld + (KV ? 0 : D) + d], a1);
      if (KV) a2 = fmaf(wp[j], dob[static_cast<size_t>(j) * D + d], a2);
    }
    if (KV) {
      go[D + d] = a1 * scale;
      go[2 * D + d] = a2;
    } else {
      go[d] = a1 * scale;
    }
  }
}

static int g_bwd_cus = 0;
static bool g_bwd_big_ok = false;

hipError_t attention_bwd_init() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  e = hipDeviceGetAttribute(&g_bwd_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e != hipSuccess) return e;
  // kernels whose LDS ring exceeds the default limit of a launch (64 KiB)
  g_bwd_big_ok = true;
  struct Big { const void *fn; int bytes; };
  const Big big[] = {
      {reinterpret_cast<const void *>(&attn_bwd_wide_bf16_kernel<false, false>), wide_lds_bytes(false)},
      {reinterpret_cast<const void *>(&attn_bwd_wide_bf16_kernel<false, true>), wide_lds_bytes(false)},
      {reinterpret_cast<const void *>(&attn_bwd_wide_bf16_kernel<true, false>), wide_lds_bytes(true)},
      {reinterpret_cast<const void *>(&attn_bwd_wide_bf16_kernel<true, true>), wide_lds_bytes(true)},
      {reinterpret_cast<const void *>(&attn_bwd_bf16_kernel<false, false, 1>), bwd256_lds_bytes(false)},
      {reinterpret_cast<const void *>(&attn_bwd_bf16_kernel<false, true, 1>), bwd256_lds_bytes(false)},
      {reinterpret_cast<const void *>(&attn_bwd_bf16_kernel<true, false, 2>), bwd256_lds_bytes(true)},
      {reinterpret_cast<const void *>(&attn_bwd_bf16_kernel<true, true, 2>), bwd256_lds_bytes(true)},
  };
  for (const Big &k : big) {
    e = hipFuncSetAttribute(k.fn, hipFuncAttributeMaxDynamicSharedMemorySize, k.bytes);
    if (e != hipSuccess) {            // not fatal: only the gradient at head dimensions 128 and 256 is refused
      (void)hipGetLastError();
      g_bwd_big_ok = false;
    }
  }
  return hipSuccess;
}

size_t tiles_attention_bwd_ws_bytes(const reslim_ctx *c, int batch, const SeqGeom *geom) {
  const size_t recs = static_cast<size_t>(batch) * c->cfg.heads * (geom ? geom->n_h : c->n_h);
  return c->cfg.dtype == RESLIM_BF16 ? align256(recs * 32) : align256(recs * 4);
}

template <bool KV, bool QS, int NSPLIT>
static hipError_t launch_bwd_256(const AttnBwdArgs &a0, hipStream_t st) {
  const int g = a0.total < g_bwd_cus ? a0.total : g_bwd_cus;    // persistent grid
  AttnBwdArgs a = a0;
  for (a.part = 0; a.part < NSPLIT; ++a.part) {
    attn_bwd_bf16_kernel<KV, QS, NSPLIT><<<dim3(g), dim3(256), bwd256_lds_bytes(KV), st>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool KV, bool QS>
static hipError_t launch_bwd_woven(const AttnBwdArgs &a0, hipStream_t st) {
  AttnBwdArgs a = a0;
  constexpr int64_t most = most_work_groups(256);
  for (int64_t first = 0; first < a.total; first += most) {
    a.first = static_cast<int>(first);
    attn_bwd_woven_bf16_kernel<KV, QS><<<dim3(static_cast<unsigned>(std::min(most, a.total - first))), dim3(256), 0, st>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Launch shapes (measured on MI355X; the file is built with MFMA operands in ordinary vector
// registers, see the build script): dh = 64: attn_bwd_woven.  dh = 128: attn_bwd_wide.
// dh = 256: dQ unsplit on 32-token blocks (15 registers spilled, still faster than two spill-free half passes), dK and dV
// together, once per half of the head's features (505 registers, no spills).  The 10B model's
// block: 6.6 ms, against 40.5 ms for unsplit dQ and dK/dV passes that spilled 130 .. 145 registers.
template <bool QS>
static hipError_t launch_bwd_all(const AttnBwdArgs &a, int dh, hipStream_t st) {
  hipError_t e;
  switch (dh) {
    case 64:
      if ((e = launch_bwd_woven<false, QS>(a, st)) != hipSuccess) return e;
      return launch_bwd_woven<true, QS>(a, st);
    case 128:
      if (!g_bwd_big_ok) return hipErrorInvalidValue;
      attn_bwd_wide_bf16_kernel<false, QS><<<dim3(min(a.total, g_bwd_cus)), dim3(256), wide_lds_bytes(false), st>>>(a);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      attn_bwd_wide_bf16_kernel<true, QS><<<dim3(min(a.total, g_bwd_cus)), dim3(256), wide_lds_bytes(true), st>>>(a);
      return hipGetLastError();
    case 256:
      if (!g_bwd_big_ok) return hipErrorInvalidValue;
      e = launch_bwd_256<false, QS, 1>(a, st);
      return e != hipSuccess ? e : launch_bwd_256<true, QS, 2>(a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_tiles_attention_bwd(const reslim_ctx *c, const void *qkv, const void *out, const float *lse,
                                      const void *dout, void *dqkv, int batch, void *ws, bool q_prescaled,
                                      hipStream_t st, const SeqGeom *geom) {
  const SeqGeom sg = geom ? *geom : ctx_geom(c);
  const int heads = c->cfg.heads, D = c->cfg.embed_dim, dh = c->dh;
  const int64_t recs = static_cast<int64_t>(batch) * heads * sg.n_h;
  if (recs == 0) return hipSuccess;
  if (c->cfg.dtype == RESLIM_BF16) {
    const float rs = 1.0f / sqrtf(static_cast<float>(dh));
    AttnBwdArgs a;
    a.qkv = static_cast<const bf16_t *>(qkv);
    a.dout = static_cast<const bf16_t *>(dout);
    a.aux = static_cast<u32x4 *>(ws);
    a.out = static_cast<const bf16_t *>(out);
    a.lse = lse;
    a.dqkv = static_cast<bf16_t *>(dqkv);
    a.tiles = sg.d_tiles;
    a.T = sg.T;
    a.heads = heads;
    a.D = D;
    a.n_h = sg.n_h;
    a.first = a.part = 0;
    a.aux_stride = recs;
    // With q pre-scaled by log2(e)/sqrt(dh) the MFMA output is the base-2 logit; the gradient with
    // respect to the UNSCALED q keeps the factor 1/sqrt(dh), the one of k becomes ln 2 (k meets the
    // scaled q).
    a.c = q_prescaled ? 1.0f : 1.4426950408889634f * rs;
    a.scq = rs;
    a.sck = q_prescaled ? 0.69314718055994531f : rs;
    a.QB = (sg.max_n_tok + 127) / 128;
    const int64_t total = static_cast<int64_t>(batch) * sg.T * heads * a.QB;
    if (total > INT32_MAX || g_bwd_cus <= 0) return hipErrorInvalidValue;
    a.total = static_cast<int>(total);
    // One work-group to a compute unit at head dimension 128: a work-group with one slot more that has a block, where others skip empty ones,
    // is waited for.  Blocks that exist are numbered instead where a fiftieth of the slots and more are empty and there are more slots than
    // compute units (16 tiles of 1128 to 1323 tokens, 24 heads: 1296 and 1201 us; of 2244 to 2448, 32 heads: 5.22 and 5.05 ms).  Finding the tile
    // takes 0.8 us a unit, more than it gives for tiles of one to three blocks (30 tokens, 1024 sets of keys: 48 and 54 us) or without empty slots
    // (1290 tokens, 16 sets: 84 and 86; 300, 256: 96 and 100), and needs a lane to a tile.
    const int64_t slots = static_cast<int64_t>(sg.T) * a.QB;
    a.per = dh == 128 && sg.T <= 64 && a.QB > 3 && total > g_bwd_cus && 50 * (slots - sg.blocks128) >= slots ? static_cast<int>(sg.blocks128) : 0;
    if (a.per) a.total = batch * heads * a.per;
    // record 0 holds -lse in the unit of the MFMA output: -lse*sqrt(dh), or -lse*log2(e) for pre-scaled q
    const float lse_f = q_prescaled ? 1.4426950408889634f : sqrtf(static_cast<float>(dh));
    a.lse_f = lse_f;
    if (dh == 256) {                       // at 64 and 128 the query-stationary launch does it
      const int64_t n_vec = static_cast<int64_t>(batch) * sg.n_h * D / 8;
      attn_bwd_prep_bf16_kernel<<<dim3(static_cast<unsigned>((n_vec + 255) / 256)), dim3(256), 0, st>>>(a.out, a.dout, lse, a.aux, n_vec, sg.n_h, heads, D, lse_f, recs);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return q_prescaled ? launch_bwd_all<true>(a, dh, st) : launch_bwd_all<false>(a, dh, st);
  }
  float *delta = static_cast<float *>(ws);
  const size_t lds = (2 * static_cast<size_t>(sg.max_n_tok) + 2 * dh) * sizeof(float);
  if (lds > 60 * 1024 || sg.n_h > INT32_MAX) return hipErrorInvalidValue;
  const int64_t n = static_cast<int64_t>(batch) * sg.n_h * heads;
  attn_bwd_delta_f32_kernel<<<dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st>>>(
      static_cast<const float *>(out), static_cast<const float *>(dout), delta, n, sg.n_h, heads, dh);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid(static_cast<unsigned>(sg.n_h), heads, batch);
  attn_bwd_f32_kernel<false><<<grid, dim3(128), lds, st>>>(static_cast<const float *>(qkv), static_cast<const float *>(dout),
                                                         lse, delta, static_cast<float *>(dqkv), sg.d_tiles,
                                                         sg.d_tile_of_tok, sg.n_h, heads, D, dh, sg.max_n_tok);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  attn_bwd_f32_kernel<true><<<grid, dim3(128), lds, st>>>(static_cast<const float *>(qkv), static_cast<const float *>(dout),
                                                        lse, delta, static_cast<float *>(dqkv), sg.d_tiles,
                                                        sg.d_tile_of_tok, sg.n_h, heads, D, dh, sg.max_n_tok);
  return hipGetLastError();
}

}  // namespace reslim
