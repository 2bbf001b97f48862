// Tile-local multi-head self-attention (ORBIT-2 Sec. 4.2): for every sample, tile
// and head, O = softmax(Q K^T / sqrt(dh)) V over the tokens of that tile only.
// The paper relies on a cache-blocked ("Flash") attention library (Sec. 4.4); the
// kernel below is written for gfx950 from the arithmetic itself.
//
// bf16 kernel.  The unit of work is 128 queries of one (sample, tile, head); each of
// the four waves of a work-group owns 32 of them.  Keys/values are visited in blocks
// of BKV rows that go from global memory straight into LDS.  Scores are computed
// TRANSPOSED, S^T = K Q^T, with MFMA 32x32x16: a lane then owns one query column
// and the softmax row statistics are in-lane reductions plus one exchange between
// the two lane halves.  The rows of the K operand are read in a permuted order
// chosen so that the accumulator registers of S^T are, without any data movement,
// the B operand (P^T) of the second MFMA, O^T = V^T P^T.  Online softmax in fp32
// with base-2 exponentials; P is rounded to bf16 for PV.  Units are numbered so the
// query blocks that share one K/V set run on one XCD (one L2).
#include <type_traits>

#include "attention_common.h"
#include "attention_plan.h"

namespace reslim {

// ------------------------------------------------------------------ bf16 kernel
// Data movement.  K and V blocks are loaded with global_load_lds_dwordx4 (no
// register staging), two stages deep with one barrier per block, both ROW-MAJOR; a
// direct load cannot pad rows, so the 16-byte chunks of a row are XOR-swizzled on
// the global-address side.  K rows use swzK (conflict-free for the 16-byte
// fragment reads, 16 lanes = 256 B per LDS cycle).  The V^T operand is read with
// ds_read_b64_tr_b16: within 16 lanes, lane i receives element i of each of the
// four 16-element rows the lanes 4r..4r+3 point at, i.e. four consecutive keys of
// feature column i -- the transpose happens in the LDS read.  Per 32 lanes that
// read touches 4 chunks of 4 consecutive rows; rows r and r+2 (dh = 64; all four
// rows at dh = 128) would hit the same banks, so V rows use their own swizzle swzV
// that moves the chunk group by row.  The address of a direct load is a
// buffer per block, made of scalars, plus a per-lane 32-bit offset that never changes.  Keys
// past the end of a ragged tile are loaded as zeros, or as its last key again (finite data; their
// probabilities are exactly zero).
//
// Softmax bookkeeping with few vector instructions per score (at dh = 64 the fp32
// vector pipe, not the matrix pipe, is the scarcer one):
//  * every S^T accumulator chain starts from `minit` = -(reference logit of this
//    lane's query), so the MFMA already delivers logit - reference;
//  * the reference is only moved (and O, L rescaled) when some query of the wave
//    meets a logit more than TAU above it -- rare after the first block -- so the
//    common block costs one max3 per three scores, one exp2 and half a convert
//    per score;
//  * the row sums L come from the bf16 probabilities the P V product uses, sixteen keys of 32
//    queries per matrix instruction of half the size (see RowSums).
// QS: the caller has already multiplied q by log2(e)/sqrt(dh) (the fused QKV
// epilogue does, before its single rounding to bf16), so the MFMA output is the
// base-2 logit itself.
//
// Scheduling.  Work-groups are PERSISTENT: the grid holds MINW work-groups per
// compute unit and each walks over its share of the units.  The K/V pipeline is
// flattened over units -- block 0 of the next unit (and its Q fragments) is in
// flight while the last block of the current one is computed.  O^T leaves the
// registers with 8-byte stores, one query row per lane (no staging, no extra
// barrier).  Measured on MI355X (c1, dh = 64): 64-key blocks with three waves per
// SIMD (156 VGPRs) beat 128-key blocks with two (0.097 vs 0.102 ms per launch).
// ST: stitched output -- a query that its tile owns writes its patch's row of a [batch, N, D]
// output, halo queries write nothing, and units or waves without an owned query are skipped (they
// still take part in the loads and barriers of their work-group).
// Row sums of the bf16 probabilities, taken from the same values the P V product uses.  The registers of P (lane l: query l % 32, eight
// keys of half l / 32) are, to v_mfma_f32_16x16x32_bf16, columns of 16 queries with queries c and c + 16 in different k; rows 0
// and 1 of `ones` pick them out.  The sum of query c ends up in register 0 of lane c, of query c + 16 in register 1 of lane c.
// It takes the matrix unit for half as long as one instruction of the P V product.  v_dot2c_f32_bf16, two probabilities an instruction
// on the vector unit, looks cheaper and is not: it does not run beside matrix instructions (two waves a SIMD, each one matrix instruction
// and then eight others: 65 ns with v_dot2c, 39 with conversions or multiplications, 33 with none).  With it a launch of 9.5M-model tiles
// took 43.8 us, 40.5 with this; 37,520 tokens of 32 heads of 128 features 1924 us and 1710.
// The zeros that keep two queries apart do so only while probabilities are finite, see reference_move.
struct RowSums {
  typedef __attribute__((ext_vector_type(4))) float f32x4;
  f32x4 v;
  __device__ __forceinline__ static bf16x8 ones(int lane) {
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = static_cast<__bf16>((lane & 15) == ((lane >> 4) & 1) ? 1.0f : 0.0f);
    return o;
  }
  __device__ __forceinline__ void reset() { v = f32x4{0.f, 0.f, 0.f, 0.f}; }
  __device__ __forceinline__ void add(const bf16x8 &ones, const bf16x8 &p) { v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, p, v, 0, 0, 0); }
  __device__ __forceinline__ void scale(float alpha) {
    v[0] *= alpha;
    v[1] *= of_next_16_lanes(alpha);
  }
  __device__ __forceinline__ float total(int lane) const {
    const float lo = __shfl(v[0], lane & 15), up = __shfl(v[1], lane & 15);
    return lane & 16 ? up : lo;
  }
};

// Head dimension 64, 32 keys of 32 queries before their exponentials (register r: key 16 (r / 8) + 8 hi + r % 8).  A query's reference is the
// largest logit of its tile's first 64 keys; of the first 32 it would be the 1 that rounding to bf16 leaves as it is for fewer queries (error of the output with logits of
// a standard deviation of 1, 64 tokens 2.08e-3 and 2.14e-3, 1290 tokens 2.317e-3 and 2.321e-3; from zero, without a first move, 1 % more with logits of 3).
// Where a later 32 keys have a logit more than kTau above some query's reference, every one of the 32 queries moves to the largest that it meets there: that
// makes the next moves rarer and leaves the largest probability at 1 more often than moves by a query's own logits alone (logits of a standard
// deviation of 9, 1290 tokens: 325 us at 512 sets of keys, error 1.683e-3; alone 341 and 1.691e-3).  The 32 are the same in the kernel with one
// query group a wave and with two, so what a query gets does not depend on the shape of the launch between these (the kernel that splits the keys over the waves has a
// reference a wave and sums in another order).
constexpr float kTau = 10.0f;            // in base-2 logits

// How a block of keys moves the references, in every bf16 kernel but the one that splits the keys over the waves.  mx: largest logit above the
// reference, of this lane's half of the keys; init: minus the reference.  limit: what logits are compared with; not a number while a query of the wave
// has met no finite logit, which keeps the reference 0 and no weight until it does (first: none has).
// A query with a logit that is +inf or not a number is lost: with the reference +inf its probabilities are 0 from here on, and 0 / 0 at the end is its row.
// They must not be what they are: times 0 they would be in the sums of the query 16 away (RowSums).  Nor does it move the others' references.
struct RefMove { float d, alpha, init; bool lost, any_lost; };
__device__ __forceinline__ RefMove reference_move(float mx, float init, const RowSums &lsum, bool first, float &limit, float tau, float c, int lane) {
  // The two lane halves exchange with v_permlane32_swap, not through LDS: an LDS lane permute makes the wave wait on the LDS counter,
  // and that wait also covers the direct-to-LDS loads just issued (measured: the prefetch stops being asynchronous).
  unsigned m_lo, m_up;
  lane_pair_exchange(__builtin_bit_cast(unsigned, mx), m_lo, m_up);
  mx = __builtin_elementwise_maximum(__builtin_bit_cast(float, m_lo), __builtin_bit_cast(float, m_up));
  RefMove m;
  m.lost = !(mx < INFINITY);
  m.any_lost = __any(m.lost);
  bool none = false;
  if (limit != limit) {
    none = first || lsum.total(lane) == 0.f;
    limit = __any(none && mx == -INFINITY && init > -INFINITY) ? __builtin_nanf("") : tau;
  }
  const float from = none ? -INFINITY : __any(mx > tau && !m.lost && !none) ? 0.f : tau;
  m.d = mx > from ? mx : 0.f;
  m.alpha = none ? 0.f : __builtin_amdgcn_exp2f(-m.d * c);
  m.init = init - m.d;
  if (__builtin_expect(m.any_lost, 0) && m.lost) {
    m.alpha = 0.f;
    m.init = -INFINITY;
  }
  return m;
}
// the scores of a lost query: everything behind them is 0
__device__ __forceinline__ void drop_lost(f32x16 &s, const RefMove &m) {
  if (__builtin_expect(m.any_lost, 0)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = m.lost ? -INFINITY : s[r];
  }
}
__device__ __forceinline__ void mask_block(f32x16 &s, int key0, int n_t, int hi) {      // keys past the tile end get -inf
#pragma unroll
  for (int r = 0; r < 16; ++r)
    if (key0 + 16 * (r / 8) + 8 * hi + (r % 8) >= n_t) s[r] = -INFINITY;
}
__device__ __forceinline__ float max3(float x, float y, float z) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(x, y), z); }
__device__ __forceinline__ float max_of_block(const f32x16 &s) {      // of this lane's half of the keys
  float m0 = max3(s[0], s[1], s[2]), m1 = max3(s[3], s[4], s[5]);
  m0 = max3(m0, s[6], s[7]); m1 = max3(m1, s[8], s[9]);
  m0 = max3(m0, s[10], s[11]); m1 = max3(m1, s[12], s[13]);
  m0 = max3(m0, s[14], s[15]);
  return __builtin_elementwise_maximum(m0, m1);
}
// A tile's first 64 keys, scores from zero
__device__ __forceinline__ void first_reference(f32x16 &s0, f32x16 &s1, f32x16 &minit, const RowSums &lsum, float &limit, float tau, float c, int lane) {
  const RefMove m = reference_move(__builtin_elementwise_maximum(max_of_block(s0), max_of_block(s1)), minit[0], lsum, true, limit, tau, c, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    s0[r] -= m.d;
    s1[r] -= m.d;
    minit[r] = m.init;
  }
  drop_lost(s0, m);
  drop_lost(s1, m);
}
// 32 later ones
__device__ __forceinline__ void move_reference(f32x16 &s, f32x16 &o0, f32x16 &o1, f32x16 &minit, RowSums &lsum, float mx, float &limit, float tau, float c, int lane) {
  const RefMove m = reference_move(mx, minit[0], lsum, false, limit, tau, c, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    s[r] -= m.d;
    minit[r] = m.init;
    o0[r] *= m.alpha;
    o1[r] *= m.alpha;
  }
  drop_lost(s, m);
  lsum.scale(m.alpha);
}

__device__ __forceinline__ unsigned lds_addr(const unsigned char *p) {
  return static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)p));
}

template <int DH, int BKV, bool QS, int MINW = 2, bool ST = false, int PQK = 1, int PPV = 1>
__global__ __launch_bounds__(256, MINW) void tiles_attention_bf16_kernel(AttnArgs a) {
  constexpr int BQ = 128;
  constexpr int ROWB = DH * 2;            // bytes per K/V row in LDS
  constexpr int CPR = DH / 8;             // 16-byte chunks per row (8 or 16)
  constexpr int RPB = 64 / CPR;           // rows per 1 KiB load block
  constexpr int TILE_B = BKV * ROWB;
  constexpr int STAGE = 2 * TILE_B;       // K block then V block
  constexpr int LPW = TILE_B / 1024 / 4;  // direct loads per wave and operand
  constexpr int NKT = BKV / 32, NKS = DH / 16, NDT = DH / 32;
  constexpr bool PIPE = DH == 64 && NKT == 2;   // second key group's softmax woven into the first group's P V
  static_assert(TILE_B % 4096 == 0 && 2 * STAGE <= 65536, "LDS plan");
  __shared__ __align__(1024) unsigned char smem[2 * STAGE];

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);   // uniform: keeps LDS destinations in scalar registers
  const int l32 = lane & 31, hi = lane >> 5;
  const int ld = 3 * a.D;
  const int G = gridDim.x;
  auto swzK = [](int r) { return CPR == 8 ? ((r & 7) ^ ((r >> 3) & 1)) : (r & 15); };
  auto swzV = [](int r) {
    return CPR == 8 ? ((((r >> 1) & 1) << 2) | (((r >> 3) & 1) << 1)) : (((r & 3) << 2) | (((r >> 3) & 1) << 1));
  };

  // ---- work units (all of this is uniform over the work-group)
  struct Unit { int n_t, q0, nkb, tile; const bf16_t *base; bf16_t *out; float *lse; };
  // stitched output: first and last query of a tile that the tile owns (its tokens are row-major
  // over the haloed box)
  auto owned_range = [&](int tile, int &lo, int &up) {
    const tile_desc &td = a.tiles[tile];
    const int bw = td.X1 - td.X0;
    lo = (td.y0 - td.Y0) * bw + (td.x0 - td.X0);
    up = (td.y1 - 1 - td.Y0) * bw + (td.x1 - 1 - td.X0);
  };
  auto decode = [&](int vb, Unit &u) -> int {      // first non-empty unit at or after vb (stride G), or >= total
    while (vb < a.total) {
      const int logical = xcd_remap_attn(vb, a.total);
      const int qb = logical % a.QB;
      int rest = logical / a.QB;
      const int head = rest % a.heads;
      rest /= a.heads;
      const int tile = rest % a.T;
      const int b = rest / a.T;
      const int n_t = a.tiles[tile].n_tok;
      bool wanted = qb * BQ < n_t;
      if constexpr (ST) {
        int lo, up;
        owned_range(tile, lo, up);
        wanted = wanted && qb * BQ <= up && qb * BQ + BQ - 1 >= lo;
      }
      if (wanted) {
        const size_t row0 = static_cast<size_t>(b) * a.n_h + a.tiles[tile].tok_off;
        u.n_t = n_t;
        u.tile = tile;
        u.q0 = qb * BQ;
        u.nkb = (n_t + BKV - 1) / BKV;
        u.base = static_cast<const bf16_t *>(a.qkv) + row0 * ld + head * DH;
        u.out = static_cast<bf16_t *>(a.out) + (ST ? static_cast<size_t>(b) * a.N : row0) * a.D + head * DH;
        u.lse = (ST || !a.lse) ? nullptr : a.lse + (static_cast<size_t>(b) * a.heads + head) * a.n_h + a.tiles[tile].tok_off;
        return vb;
      }
      vb += G;
    }
    return vb;
  };
  Unit cur, nxt;
  int vb = decode(blockIdx.x, cur);
  if (vb >= a.total) return;
  // stitched output: a wave whose 32 queries are all halo copies does no arithmetic
  bool wave_owns = true;
  auto set_wave_owns = [&]() {
    if constexpr (ST) {
      int lo, up;
      owned_range(cur.tile, lo, up);
      const int wq0 = cur.q0 + wave * 32;
      wave_owns = wq0 <= up && wq0 + 31 >= lo;
    }
  };
  set_wave_owns();
  vb = decode(vb + G, nxt);
  bool has_next = vb < a.total;

  // ---- load side: lane -> (row of the block, 16-byte chunk), per-lane byte offsets
  unsigned offK[LPW], offV[LPW];
  const int ld2 = ld * 2;
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int r = (wave + 4 * i) * RPB + lane / CPR;
    offK[i] = r * ld2 + ((lane % CPR) ^ swzK(r)) * 16;
    offV[i] = r * ld2 + ((lane % CPR) ^ swzV(r)) * 16 + a.D * 2;
  }
  // The buffer covers exactly the rows of a block that exist, from the head's keys on: rows past the tile's end are loaded as zeros, or, at head dimensions 128 and 256, are
  // its last row again (1024 sets of keys of 100 tokens 24.4 us, 26.3 with zeros, which take no access but more time; of 40 tokens 12.1 and 12.4; at dimension 64 the same).
  auto issue = [&](const Unit &u, int kv0, int buf) {
    unsigned char *sk = smem + buf * STAGE;
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(u.base + a.D + static_cast<size_t>(kv0) * ld), 0,
                                                                         min(u.n_t - kv0, BKV) * ld2 - 2 * a.D, 0x00020000);
    auto load = [&](int i, int back) __attribute__((always_inline)) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (__attribute__((address_space(3))) void *)(sk + (wave + 4 * i) * 1024), 16, static_cast<int>(offK[i]) - back, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (__attribute__((address_space(3))) void *)(sk + TILE_B + (wave + 4 * i) * 1024), 16, static_cast<int>(offV[i]) - back, 0, 0, 0);
    };
    const int lim = u.n_t - 1 - kv0;     // last row of the block that exists
    if (DH >= 128 && lim < BKV - 1) {      // uniform
#pragma unroll
      for (int i = 0; i < LPW; ++i) load(i, max((wave + 4 * i) * RPB + lane / CPR - lim, 0) * ld2);
    } else {
#pragma unroll
      for (int i = 0; i < LPW; ++i) load(i, 0);
    }
  };
  bf16x8 qf[NKS];
  auto load_q = [&](const Unit &u) {
    const int qrow = min(u.q0 + wave * 32 + l32, u.n_t - 1);
    const bf16_t *qp = u.base + static_cast<size_t>(qrow) * ld + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qp + ks * 16);
  };

  // ---- read side
  // K fragment: A-operand row l32 carries key key_perm(l32) of its 32-key group.
  // V^T fragment through the transposing read: this lane points at key row
  // 8*hi + 4*e + (lane%16)/4 of a 16-key step and at the 4 features
  // 32*dt + 16*((lane/16)&1) + 4*(lane%4) .. +3
  const int kr = key_perm(l32);
  const int k_row = kr * ROWB, k_swz = swzK(kr);
  const int L16 = lane & 15;
  int v_addr[2][NDT];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int vr = 8 * hi + 4 * e + (L16 >> 2);
#pragma unroll
    for (int d = 0; d < NDT; ++d) {
      const int o = 32 * d + 16 * ((lane >> 4) & 1) + 4 * (L16 & 3);
      v_addr[e][d] = TILE_B + vr * ROWB + (((o >> 3) ^ swzV(vr)) << 4) + ((o >> 2) & 1) * 8;
    }
  }

  f32x16 o[NDT], minit;
  RowSums lsum;
  const bf16x8 ones = RowSums::ones(lane);
  const float c = QS ? 1.0f : a.scale_log2;     // MFMA output -> base-2 logit
  const float TAU = kTau / c;                     // in units of the MFMA output
  float limit;                                    // TAU, or not a number (reference_move)
  auto reset = [&]() {
#pragma unroll
    for (int d = 0; d < NDT; ++d)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) minit[r] = 0.f;
    lsum.reset();
    limit = __builtin_nanf("");
  };
  reset();
  load_q(cur);
  issue(cur, 0, 0);

  int kb = 0;
  for (int g = 0;; ++g) {
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0): this wave's loads of block g (and earlier stores) are done
    __syncthreads();                        // ... and everybody's; the other buffer is free
    const bool last = kb + 1 == cur.nkb;
    if (!last) issue(cur, (kb + 1) * BKV, (g + 1) & 1);
    else if (has_next) issue(nxt, 0, (g + 1) & 1);
    const unsigned char *st = smem + (g & 1) * STAGE;
    const int kv0 = kb * BKV;
    const bool active = cur.q0 + wave * 32 < cur.n_t && wave_owns;   // wave-uniform

    f32x16 s[NKT];
    const unsigned k_at = lds_addr(st) + k_row + ((hi ^ k_swz) << 4);
    // scores of 32 or 64 keys at head dimension 64, every fragment requested ahead of the products (from one address: four would be four registers more)
    auto score_groups = [&](auto first_c, auto count_c) __attribute__((always_inline)) {
      constexpr int FIRST = decltype(first_c)::value, COUNT = decltype(count_c)::value;
      bf16x8 kf[COUNT][NKS];
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int i = 0; i < COUNT; ++i) kf[i][ks] = *reinterpret_cast<__attribute__((address_space(3))) bf16x8 *>((k_at ^ (ks * 32)) + (FIRST + i) * 32 * ROWB);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
        for (int i = 0; i < COUNT; ++i) s[FIRST + i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i][ks], qf[ks], ks == 0 ? minit : s[FIRST + i], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    if (active) {
      // The MFMA phases run at raised wave priority, the softmax arithmetic at the default one: a
      // wave whose operands are ready gets the matrix pipe ahead of the vector work of the other
      // waves on its SIMD (c1, same box: 0.0882 -> 0.0862 ms; no effect on the gradient kernels or
      // the GEMMs, where it was tried too).  At dh = 64 the two phases get DIFFERENT levels (scores
      // 2, P V 1; c3 shapes, same box: 3.47-3.51 ms with 1 / 1, 3.43-3.44 with 2 / 1, 1 / 2 or
      // 3 / 1, 3.50 with 2 / 2, 3.62 with the P V phase at the default level, 3.76 with none).
      __builtin_amdgcn_s_setprio(PQK);
      // feature step outermost: consecutive MFMAs belong to different accumulator chains
      if constexpr (PIPE) {
        score_groups(I0{}, I2{});
      } else if constexpr (DH <= 128) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
          for (int kt = 0; kt < NKT; ++kt) {
            const bf16x8 kf = *reinterpret_cast<const bf16x8 *>(st + kt * 32 * ROWB + k_row + (((2 * ks + hi) ^ k_swz) << 4));
            s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], ks == 0 ? minit : s[kt], 0, 0, 0);
          }
        }
      } else {
        // dh = 256 runs one wave per SIMD: the fragment reads go PF steps ahead of the MFMAs that
        // use them (ring of PF + 1 register sets; a scheduling barrier per step keeps that order),
        // so a wave hides its own LDS latency (1.87 -> 1.75 ms for the 10B model's block; with the
        // two waves per SIMD of dh = 128 the same ring gains nothing)
        constexpr int PF = 2, NSTEP = NKS * NKT;
        bf16x8 kf[PF + 1];
        auto fetch = [&](int i) {
          const int ks = i / NKT, kt = i % NKT;
          kf[i % (PF + 1)] = *reinterpret_cast<const bf16x8 *>(st + kt * 32 * ROWB + k_row + (((2 * ks + hi) ^ k_swz) << 4));
        };
#pragma unroll
        for (int i = 0; i < PF; ++i) fetch(i);
#pragma unroll
        for (int i = 0; i < NSTEP; ++i) {
          if (i + PF < NSTEP) fetch(i + PF);
          const int ks = i / NKT, kt = i % NKT;
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i % (PF + 1)], qf[ks], ks == 0 ? minit : s[kt], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    bool woven = true;
    if constexpr (PIPE) {
      if (active) {
        // The first block's 64 keys give the references; later ones move at a group of 32 keys, by the group's logits, and the scores behind start from where they went:
        // where they move at the first group the second's are computed once more.  One branch for both, which the first block of every tile takes, so what it costs is
        // the smallest launches' time (1 token, 256 sets of keys 4.16 us; 4.80 with the first 32 keys' references, the second group's scores again and each V fragment waited for by
        // itself).  Logits of a standard deviation of 0.3, 3 and 9: 400 tokens, 64 sets 11.4, 11.7 and 14.2 us, 1290 tokens 40.1, 41.7 and 49.3.
        const bool ragged = kv0 + BKV > cur.n_t;
        if (ragged) {
          mask_block(s[0], kv0, cur.n_t, hi);
          mask_block(s[1], kv0 + 32, cur.n_t, hi);
        }
        const float m0 = max_of_block(s[0]), m01 = __builtin_elementwise_maximum(m0, max_of_block(s[1]));
        if (__any(!(m01 <= limit))) {
          const bool first = kb == 0;
          woven = first;
          if (first || __any(!(m0 <= limit))) {
            const RefMove m = reference_move(first ? m01 : m0, minit[0], lsum, first, limit, TAU, c, lane);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              s[0][r] -= m.d;
              o[0][r] *= m.alpha;
              o[1][r] *= m.alpha;
              minit[r] = m.init;
            }
            lsum.scale(m.alpha);
            drop_lost(s[0], m);
            if (first) {
#pragma unroll
              for (int r = 0; r < 16; ++r) s[1][r] -= m.d;
              drop_lost(s[1], m);
            } else {
              score_groups(I1{}, I1{});
              if (ragged) mask_block(s[1], kv0 + 32, cur.n_t, hi);
              woven = !__any(!(max_of_block(s[1]) <= limit));      // no reference moves at the second group
            }
          }
        }
        if (!woven) {
          // One group after the other.  Same operations in the same order as below, and as in the kernel with two query groups: same bits.
          const unsigned va = lds_addr(st) + static_cast<unsigned>(v_addr[0][0]);
          auto group = [&](auto kt_c) __attribute__((always_inline)) {
            constexpr int kt = decltype(kt_c)::value;
            VFrag64 vf;
            v_frag_issue<kt * 32 * ROWB>(vf, va);
            bf16x8 pf[2];
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
              for (int e = 0; e < 8; ++e) pf[h2][e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(QS ? s[kt][8 * h2 + e] : s[kt][8 * h2 + e] * c));
            v_frag_wait(vf);
#pragma unroll
            for (int h2 = 0; h2 < 2; ++h2) {
              lsum.add(ones, pf[h2]);
#pragma unroll
              for (int d = 0; d < 2; ++d) {
                typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
                const u64x2 both = {vf.r[h2][d][0], vf.r[h2][d][1]};
                o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf[h2], o[d], 0, 0, 0);
              }
            }
          };
          group(std::integral_constant<int, 0>{});
          move_reference(s[1], o[0], o[1], minit, lsum, max_of_block(s[1]), limit, TAU, c, lane);
          group(std::integral_constant<int, 1>{});
        }
      }
    }
    // the query fragments are dead after the last block of a unit: fetch the next unit's
    if (last && has_next) load_q(nxt);
    if (active) {
      if constexpr (!PIPE) {
        if (kv0 + BKV > cur.n_t) {           // ragged last block: keys past the tile end get -inf
#pragma unroll
          for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
              const int key = kv0 + kt * 32 + 16 * (r / 8) + 8 * hi + (r % 8);
              if (key >= cur.n_t) s[kt][r] = -INFINITY;
            }
        }
        float mx = max_of_block(s[0]);
#pragma unroll
        for (int kt = 1; kt < NKT; ++kt) mx = __builtin_elementwise_maximum(mx, max_of_block(s[kt]));
        if (__any(!(mx <= limit))) {
          const RefMove m = reference_move(mx, minit[0], lsum, kb == 0, limit, TAU, c, lane);
#pragma unroll
          for (int kt = 0; kt < NKT; ++kt) {
#pragma unroll
            for (int r = 0; r < 16; ++r) s[kt][r] -= m.d;
            drop_lost(s[kt], m);
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) minit[r] = m.init;
          if (kb != 0) {
#pragma unroll
            for (int dd = 0; dd < NDT; ++dd)
#pragma unroll
              for (int r = 0; r < 16; ++r) o[dd][r] *= m.alpha;
            lsum.scale(m.alpha);
          }
        }
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            s[kt][r] = __builtin_amdgcn_exp2f(QS ? s[kt][r] : s[kt][r] * c);
      }
      __builtin_amdgcn_s_setprio(PPV);
      if constexpr (PIPE) {
        if (woven) {
        // The exponentials and conversions of the second 32-key group are placed between the
        // matrix instructions of the first group's P V product: a wave issues in order, so its own
        // vector work only overlaps its matrix work when the two are interleaved in the stream.
        const unsigned va = lds_addr(st) + static_cast<unsigned>(v_addr[0][0]);
        typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
        // the first group's V reads are issued ahead of its exponentials, which cover their latency
        VFrag64 vf0, vf1;
        v_frag_issue<0>(vf0, va);
#pragma unroll
        for (int r = 0; r < 16; ++r) s[0][r] = __builtin_amdgcn_exp2f(QS ? s[0][r] : s[0][r] * c);
        bf16x8 pf0[2], pf1[2];
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
          for (int e = 0; e < 8; ++e) pf0[h2][e] = static_cast<__bf16>(s[0][8 * h2 + e]);
        v_frag_wait(vf0);
        v_frag_issue<32 * ROWB>(vf1, va);     // in flight under the whole first group
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          lsum.add(ones, pf0[h2]);
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const u64x2 both = {vf0.r[h2][d][0], vf0.r[h2][d][1]};
            o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf0[h2], o[d], 0, 0, 0);
          }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) s[1][r] = __builtin_amdgcn_exp2f(QS ? s[1][r] : s[1][r] * c);
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
          for (int e = 0; e < 8; ++e) pf1[h2][e] = static_cast<__bf16>(s[1][8 * h2 + e]);
        // one matrix instruction, then six vector instructions, four times (16 exponentials + 8 conversions)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        v_frag_wait(vf1);
#pragma unroll
        for (int h2 = 0; h2 < 2; ++h2) {
          lsum.add(ones, pf1[h2]);
#pragma unroll
          for (int d = 0; d < 2; ++d) {
            const u64x2 both = {vf1.r[h2][d][0], vf1.r[h2][d][1]};
            o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf1[h2], o[d], 0, 0, 0);
          }
        }
        }
      } else if constexpr (DH == 64) {
        // LDS byte addresses of this lane's four fragment pointers in the current stage
        const unsigned st_off = static_cast<unsigned>(reinterpret_cast<uintptr_t>(
            (__attribute__((address_space(3))) const unsigned char *)st));
        unsigned va[2][2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int d = 0; d < 2; ++d) va[e][d] = st_off + static_cast<unsigned>(v_addr[e][d]);
        auto group = [&](auto kt_c) {
          constexpr int kt = decltype(kt_c)::value;
          VFrag64 vf;
          v_frag_issue<kt * 32 * ROWB>(vf, va);
          bf16x8 pf[2];
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[h2][e] = static_cast<__bf16>(s[kt][8 * h2 + e]);
          v_frag_wait(vf);
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2) {
            lsum.add(ones, pf[h2]);
#pragma unroll
            for (int d = 0; d < 2; ++d) {
              typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
              const u64x2 both = {vf.r[h2][d][0], vf.r[h2][d][1]};
              o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf[h2], o[d], 0, 0, 0);
            }
          }
        };
        group(std::integral_constant<int, 0>{});
        group(std::integral_constant<int, 1>{});
        if constexpr (NKT == 4) {
          group(std::integral_constant<int, 2>{});
          group(std::integral_constant<int, 3>{});
        }
      } else if constexpr (DH <= 128) {
#pragma unroll
        for (int kt = 0; kt < NKT; ++kt) {
#pragma unroll
          for (int h2 = 0; h2 < 2; ++h2) {
            bf16x8 pf;
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[e] = static_cast<__bf16>(s[kt][8 * h2 + e]);
            lsum.add(ones, pf);
#pragma unroll
            for (int d = 0; d < NDT; ++d) {
              const unsigned char *vp = st + (kt * 32 + h2 * 16) * ROWB;
              const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                  (s16x4 __attribute__((address_space(3))) *)(vp + v_addr[0][d]));
              const s16x4 hi4 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                  (s16x4 __attribute__((address_space(3))) *)(vp + v_addr[1][d]));
              typedef __attribute__((ext_vector_type(8))) short s16x8;
              const s16x8 both = __builtin_shufflevector(lo, hi4, 0, 1, 2, 3, 4, 5, 6, 7);
              const bf16x8 vf = __builtin_bit_cast(bf16x8, both);
              o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf, o[d], 0, 0, 0);
            }
          }
        }
      } else {
        // the same ring for the transposed V fragments of P V: step = (key group, half, feature block)
        constexpr int PF = 2, NSTEP = NKT * 2 * NDT;
        typedef __attribute__((ext_vector_type(8))) short s16x8;
        s16x4 vlo[PF + 1], vhi[PF + 1];
        auto fetch = [&](int i) {
          const int d = i % NDT, h2 = (i / NDT) % 2, kt = i / (2 * NDT);
          const unsigned char *vp = st + (kt * 32 + h2 * 16) * ROWB;
          vlo[i % (PF + 1)] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(vp + v_addr[0][d]));
          vhi[i % (PF + 1)] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)(vp + v_addr[1][d]));
        };
#pragma unroll
        for (int i = 0; i < PF; ++i) fetch(i);
        bf16x8 pf;
#pragma unroll
        for (int i = 0; i < NSTEP; ++i) {
          if (i + PF < NSTEP) fetch(i + PF);
          const int d = i % NDT, h2 = (i / NDT) % 2, kt = i / (2 * NDT);
          if (d == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) pf[e] = static_cast<__bf16>(s[kt][8 * h2 + e]);
            lsum.add(ones, pf);
          }
          const s16x8 both = __builtin_shufflevector(vlo[i % (PF + 1)], vhi[i % (PF + 1)], 0, 1, 2, 3, 4, 5, 6, 7);
          o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf, o[d], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
    __builtin_amdgcn_s_setprio(0);
    if (!last) { ++kb; continue; }

    // ---- end of a unit: normalise and store this lane's query row, then move on
    const int qrow = cur.q0 + wave * 32 + l32;
    int orow = qrow;
    bool keep = true;
    if constexpr (ST) {                    // the query's patch, if this tile owns it
      const tile_desc &td = a.tiles[cur.tile];
      const int bw = td.X1 - td.X0;
      const int yy = td.Y0 + qrow / bw, xx = td.X0 + qrow % bw;
      keep = yy >= td.y0 && yy < td.y1 && xx >= td.x0 && xx < td.x1;
      orow = yy * a.Wp + xx;
    }
    if (active && qrow < cur.n_t) {
      const float ltot = lsum.total(lane);
      const float inv = 1.0f / ltot;
      // log-sum-exp of the logits (kept for the gradient): reference + log of the sum
      if (!ST && cur.lse && hi == 0) cur.lse[qrow] = (__builtin_amdgcn_logf(ltot) - minit[0] * c) * 0.69314718055994531f;
      bf16_t *op = cur.out + static_cast<size_t>(orow) * a.D + hi * 4;
      if (keep) {
#pragma unroll
        for (int d = 0; d < NDT; ++d)
#pragma unroll
          for (int r4 = 0; r4 < 4; ++r4) {
            // registers 4*r4 .. 4*r4+3 hold features 32d + 8*r4 + 4*hi + (0..3) of query l32
            bf16x4 tmp;
#pragma unroll
            for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(o[d][4 * r4 + e] * inv);
            *reinterpret_cast<u32x2 *>(op + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
          }
      }
    }
    if (!has_next) break;
    cur = nxt;
    set_wave_owns();
    vb = decode(vb + G, nxt);
    has_next = vb < a.total;
    kb = 0;
    reset();
  }
}

// ------------------------------------------------------------------ bf16 kernel at head dimension 64: two query groups a wave
// The kernel above spends the matrix instructions' time plus the vector instructions' time: a wave issues in order, so its softmax runs
// beside its own matrix instructions only where the two are woven, and there the scores and the last quarter of P V are not.  Here a
// wave has two groups of 32 queries, A and B, and every phase of 32 keys weaves the matrix instructions of one (scores of the next
// block, P V of the last) with the softmax of the other:
//   phase 0: S_A(i + 1), O_A += V(i) P_A(i)  beside the softmax of S_B(i);   phase 1: S_B(i + 1), O_B += V(i) P_B(i)  beside that of S_A(i + 1)
// The first two blocks' scores come first: their largest is the reference.
// Fragments of K and V are read from LDS once for both.  Order within a phase is pinned, one matrix instruction and what fits beside it
// at a time (scheduling barriers; the empty statements keep the compiler from sinking vector work out of its place).
// A block of 32 keys is 8 KiB; four lie in LDS, two of them in flight (five to ten took the same time).  K fragments of block i + 2 are read as soon as
// block i + 1's last have been used, V's behind the first scores, so only the barrier in the middle (block i + 2 has landed, block i is
// free) and the rare change of a reference stand between the phases; loads are issued between the scores of phase 1.
// Same operations in the same order on every query as in the kernel above, whose launches it shares: same bits.
// What bounds it: matrix pipe and vector unit are each busy about half of the time at 1.9 GHz, and every part costs its power: without
// the loads a launch takes 0.89 of its time, without the exponentials 0.95.  403,200 tokens of 16 heads in tiles of 1274 to 1643: 3.06 ms with the kernel
// above, 2.71 here (815 and 920 TFLOP/s); 42,560 of 8 in tiles of 612 to 720 89.8 us and 83.5.  When it is taken: attention_plan.h.
template <bool QS, bool ST, int NW>
__global__ __launch_bounds__(64 * NW, 2) void tiles_attention_pair_bf16_kernel(AttnArgs a) {
  constexpr int DH = 64, ROWB = DH * 2, TILE = 32 * ROWB, STAGE = 2 * TILE, NST = 4, NKS = DH / 16;
  constexpr int BQ = 64 * NW, LPO = 4 / NW;            // direct loads of a wave per block and operand
  __shared__ __align__(1024) unsigned char smem[NST * STAGE];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int ld = 3 * a.D, ld2 = ld * 2;
  const int logical = xcd_remap_attn(blockIdx.x, a.total);
  const int qb = logical % a.QB;
  int rest = logical / a.QB;
  const int head = rest % a.heads;
  rest /= a.heads;
  const int tile = rest % a.T, b = rest / a.T;
  const tile_desc &td = a.tiles[tile];
  const int n_t = td.n_tok, q0 = qb * BQ, wq0 = q0 + wave * 64;
  if (q0 >= n_t) return;                               // uniform
  const int bw = td.X1 - td.X0;
  bool active = wq0 < n_t;
  if constexpr (ST) {                                  // first and last query that the tile owns
    const int lo = (td.y0 - td.Y0) * bw + (td.x0 - td.X0), up = (td.y1 - 1 - td.Y0) * bw + (td.x1 - 1 - td.X0);
    if (q0 > up || q0 + BQ - 1 < lo) return;
    active = active && wq0 <= up && wq0 + 63 >= lo;
  }
  const int64_t row0 = static_cast<int64_t>(b) * a.n_h + td.tok_off;
  const bf16_t *const base = static_cast<const bf16_t *>(a.qkv) + row0 * ld + head * DH;
  const int nkb = (n_t + 31) / 32;

  // ---- load side
  auto swzK = [](int r) { return (r & 7) ^ ((r >> 3) & 1); };
  auto swzV = [](int r) { return (((r >> 1) & 1) << 2) | (((r >> 3) & 1) << 1); };
  unsigned offK[LPO], offV[LPO];
#pragma unroll
  for (int i = 0; i < LPO; ++i) {
    const int r = (wave + NW * i) * 8 + lane / 8;
    offK[i] = r * ld2 + ((lane % 8) ^ swzK(r)) * 16;
    offV[i] = r * ld2 + ((lane % 8) ^ swzV(r)) * 16 + a.D * 2;
  }
  auto after = [](unsigned stage) { return stage == (NST - 1) * STAGE ? 0u : stage + STAGE; };
  // The buffer covers exactly the rows of one block that exist, from the head's keys on: rows past the tile's end and blocks past the
  // last one are loaded as zeros without an access.
  const bf16_t *k_ptr = base + a.D;
  int rows_left = n_t;
  unsigned l_stage = 0;
  __amdgpu_buffer_rsrc_t rows;
  auto next_block = [&]() {
    rows = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(k_ptr), 0, max(min(rows_left, 32) * ld2 - 2 * a.D, 0), 0x00020000);
    k_ptr += static_cast<size_t>(32) * ld;
    rows_left -= 32;
  };
  auto load_keys = [&]() {
#pragma unroll
    for (int i = 0; i < LPO; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (__attribute__((address_space(3))) void *)(smem + l_stage + (wave + NW * i) * 1024), 16,
                                               static_cast<int>(offK[i]), 0, 0, 0);
  };
  auto load_values = [&]() {
#pragma unroll
    for (int i = 0; i < LPO; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rows, (__attribute__((address_space(3))) void *)(smem + l_stage + TILE + (wave + NW * i) * 1024), 16,
                                               static_cast<int>(offV[i]), 0, 0, 0);
    l_stage = after(l_stage);
  };
  auto load_block = [&]() {
    next_block();
    load_keys();
    load_values();
  };
  // all but the youngest NST - 3 blocks of this wave's loads are done, then everybody's
  auto landed = [&]() {
    constexpr int N = 2 * LPO * (NST - 3);
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4 << 14));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };

  bf16x8 q[2][NKS];
  if (active) {
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      const bf16_t *qp = base + static_cast<size_t>(min(wq0 + 32 * g + l32, n_t - 1)) * ld + hi * 8;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) q[g][ks] = *reinterpret_cast<const bf16x8 *>(qp + ks * 16);
    }
  }
  for (int i = 0; i < NST - 1; ++i) load_block();
  landed();                              // blocks 0 and 1
  load_block();
  if (!active) {                         // loads and barriers only
    for (int i = 0; i + 1 < nkb; ++i) {
      landed();
      load_block();
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // no load into LDS outlives its work-group
    return;
  }

  // ---- read side
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)smem));
  const int kr = key_perm(l32);
  const unsigned k_base = lds0 + kr * ROWB + ((hi ^ swzK(kr)) << 4);
  const int vr = 8 * hi + ((lane & 15) >> 2), vo = 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  const unsigned v_base = lds0 + TILE + vr * ROWB + (((vo >> 3) ^ swzV(vr)) << 4) + ((vo >> 2) & 1) * 8;
  bf16x8 kf[NKS];
  unsigned k_stage = 0, v_stage = 0;
  auto read_k = [&]() __attribute__((always_inline)) {
    const unsigned at = k_base + k_stage;
    k_stage = after(k_stage);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) kf[ks] = *reinterpret_cast<__attribute__((address_space(3))) bf16x8 *>(at ^ (ks * 32));
  };
  VFrag64 vf;
  auto issue_v = [&]() __attribute__((always_inline)) {
    const unsigned at = v_base + v_stage;
    v_stage = after(v_stage);
    v_frag_issue<0>(vf, at);
  };

  const float c = QS ? 1.0f : a.scale_log2;     // MFMA output -> base-2 logit
  const float TAU = kTau / c;                     // in units of the MFMA output
  float limit[2] = {__builtin_nanf(""), __builtin_nanf("")};      // TAU, or not a number (reference_move)
  f32x16 s[2], o[2][2], minit[2];
  bf16x8 p[2][2];
  RowSums lsum[2];
  lsum[0].reset();
  lsum[1].reset();
  const bf16x8 ones = RowSums::ones(lane);
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      minit[g][r] = 0.f;
      o[g][0][r] = 0.f;
      o[g][1][r] = 0.f;
    }
  auto score = [&](auto g_c, auto ks_c) __attribute__((always_inline)) {
    constexpr int g = decltype(g_c)::value, ks = decltype(ks_c)::value;
    if constexpr (ks == 0) {               // the empty statements: from minit in its place, without a copy of it
      asm volatile("" : "+v"(minit[g]));
      s[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[0], q[g][0], minit[g], 0, 0, 0);
      asm volatile("" : "+v"(s[g]), "+v"(minit[g]));
    }
    else s[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], q[g][ks], s[g], 0, 0, 0);
  };
  auto value = [&](auto g_c, auto i_c) __attribute__((always_inline)) {        // i: half of the keys, block of features
    constexpr int g = decltype(g_c)::value, h2 = decltype(i_c)::value / 2, d = decltype(i_c)::value % 2;
    typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
    const u64x2 both = {vf.r[h2][d][0], vf.r[h2][d][1]};
    o[g][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), p[g][h2], o[g][d], 0, 0, 0);
  };
  auto exps = [&](auto g_c, auto r_c) __attribute__((always_inline)) {         // four values
    constexpr int g = decltype(g_c)::value, r = decltype(r_c)::value;
    float e0 = __builtin_amdgcn_exp2f(QS ? s[g][r] : s[g][r] * c), e1 = __builtin_amdgcn_exp2f(QS ? s[g][r + 1] : s[g][r + 1] * c);
    float e2 = __builtin_amdgcn_exp2f(QS ? s[g][r + 2] : s[g][r + 2] * c), e3 = __builtin_amdgcn_exp2f(QS ? s[g][r + 3] : s[g][r + 3] * c);
    asm volatile("" : "+v"(e0), "+v"(e1), "+v"(e2), "+v"(e3));
    s[g][r] = e0; s[g][r + 1] = e1; s[g][r + 2] = e2; s[g][r + 3] = e3;
  };
  auto convert = [&](auto g_c, auto h_c) __attribute__((always_inline)) {
    constexpr int g = decltype(g_c)::value, h2 = decltype(h_c)::value;
#pragma unroll
    for (int e = 0; e < 8; ++e) p[g][h2][e] = static_cast<__bf16>(s[g][8 * h2 + e]);
    asm volatile("" : "+v"(p[g][h2]));
  };
  auto add_up = [&](auto g_c, auto h_c) __attribute__((always_inline)) {
    constexpr int g = decltype(g_c)::value, h2 = decltype(h_c)::value;
    lsum[g].add(ones, p[g][h2]);
  };
  auto fence = []() { __builtin_amdgcn_sched_barrier(0); };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  typedef std::integral_constant<int, 2> I2;
  typedef std::integral_constant<int, 3> I3;
  typedef std::integral_constant<int, 4> I4;
  typedef std::integral_constant<int, 8> I8;
  typedef std::integral_constant<int, 12> I12;
  // One phase: matrix instructions of group gm (scores of a block where qk is 2, P V of the block before where pv) with the softmax of block
  // blk of the other group between them; with qk of 1 and 2 the loads that go with it.  known: the references are what these scores gave.
  auto phase = [&](auto gm, auto qk, auto pv, auto known, int blk) __attribute__((always_inline)) {
    constexpr int GM = decltype(gm)::value, GS = 1 - GM;
    constexpr bool QK = decltype(qk)::value == 2, LD = decltype(qk)::value >= 1 && GM == 1, PV = decltype(pv)::value, NEW = !decltype(known)::value;
    std::integral_constant<int, GS> gs;
    f32x16 &x = s[GS];
    if (NEW && __builtin_expect(blk * 32 + 32 > n_t, 0)) mask_block(x, blk * 32, n_t, hi);
    if constexpr (QK) score(gm, I0{});
    fence();
    if constexpr (LD) { next_block(); load_keys(); }
    if constexpr (PV && GM == 0) issue_v();
    float m0 = max3(x[0], x[1], x[2]), m1 = max3(x[3], x[4], x[5]);
    m0 = max3(m0, x[6], x[7]); m1 = max3(m1, x[8], x[9]);
    fence();
    if constexpr (QK) score(gm, I1{});
    fence();
    if constexpr (LD) load_values();
    m0 = max3(m0, x[10], x[11]); m1 = max3(m1, x[12], x[13]);
    m0 = max3(m0, x[14], x[15]);
    const float mx = __builtin_elementwise_maximum(m0, m1);
    if (NEW && __builtin_expect(__any(!(mx <= limit[GS])), 0)) move_reference(x, o[GS][0], o[GS][1], minit[GS], lsum[GS], mx, limit[GS], TAU, c, lane);
    fence();
    if constexpr (QK) score(gm, I2{});
    fence();
    exps(gs, I0{});
    fence();
    if constexpr (QK) score(gm, I3{});
    fence();
    if constexpr (LD) read_k();                  // of the block after; past the last one zeros
    exps(gs, I4{});
    if constexpr (PV && GM == 0) v_frag_wait(vf);
    fence();
    if constexpr (PV) value(gm, I0{});
    fence();
    exps(gs, I8{});
    fence();
    if constexpr (PV) add_up(gm, I0{});
    if constexpr (PV) value(gm, I1{});
    fence();
    exps(gs, I12{});
    fence();
    if constexpr (PV) value(gm, I2{});
    fence();
    convert(gs, I0{});
    fence();
    if constexpr (PV) value(gm, I3{});
    fence();
    convert(gs, I1{});
    fence();
    if constexpr (PV) add_up(gm, I1{});
    fence();
  };
  typedef std::true_type Yes;
  typedef std::false_type No;

  // The first two blocks' scores, from zero, give the references; the second's stay where the outputs will be.
  f32x16 second[2];
  auto scores = [&](f32x16 &x, int g) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], q[g][ks], ks == 0 ? minit[g] : x, 0, 0, 0);
  };
  read_k();
  scores(s[0], 0);
  scores(s[1], 1);
  read_k();
  scores(second[0], 0);
  scores(second[1], 1);
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    if (n_t < 32) mask_block(s[g], 0, n_t, hi);
    if (n_t < 64) mask_block(second[g], 32, n_t, hi);
    first_reference(s[g], second[g], minit[g], lsum[g], limit[g], TAU, c, lane);
  }
  typedef std::integral_constant<int, 0> None;
  typedef std::integral_constant<int, 1> Loads;
  typedef std::integral_constant<int, 2> Scores;
  phase(I1{}, None{}, No{}, Yes{}, 0);
  if (nkb > 1) {
    s[0] = second[0];
    phase(I0{}, None{}, Yes{}, Yes{}, 0);
    s[1] = second[1];
    landed();                            // block 2; everybody has left block 0, whose place takes block NST
    phase(I1{}, Loads{}, Yes{}, Yes{}, 1);
  }
#pragma unroll 1
  for (int i = 1; i + 1 < nkb; ++i) {
    phase(I0{}, Scores{}, Yes{}, No{}, i);
    landed();                            // block i + 2; everybody has left block i, whose place takes block i + NST
    phase(I1{}, Scores{}, Yes{}, No{}, i + 1);
  }
  phase(I0{}, None{}, Yes{}, No{}, nkb - 1);
  value(I1{}, I0{}); value(I1{}, I1{}); value(I1{}, I2{}); value(I1{}, I3{});
  add_up(I1{}, I0{});
  add_up(I1{}, I1{});

  if constexpr (ST) asm volatile("" : : "v"(minit[0][0]), "v"(minit[1][0]));      // alive to the end as for the log-sum-exp: it spills otherwise
  __builtin_amdgcn_s_waitcnt(0x0F70);    // no load into LDS outlives its work-group

  // ---- normalise and store this lane's two query rows
  float *const lse = (ST || !a.lse) ? nullptr : a.lse + (static_cast<size_t>(b) * a.heads + head) * a.n_h + td.tok_off;
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int qrow = wq0 + 32 * g + l32;
    int64_t orow = row0 + qrow;
    bool keep = qrow < n_t;
    if constexpr (ST) {                  // the query's patch, if this tile owns it
      const int yy = td.Y0 + qrow / bw, xx = td.X0 + qrow % bw;
      keep = keep && yy >= td.y0 && yy < td.y1 && xx >= td.x0 && xx < td.x1;
      orow = static_cast<int64_t>(b) * a.N + static_cast<int64_t>(yy) * a.Wp + xx;
    }
    const float ltot = lsum[g].total(lane);
    const float inv = 1.0f / ltot;
    if (!ST && lse && hi == 0 && keep) lse[qrow] = (__builtin_amdgcn_logf(ltot) - minit[g][0] * c) * 0.69314718055994531f;
    if (keep) {
      bf16_t *op = static_cast<bf16_t *>(a.out) + orow * a.D + head * DH + hi * 4;
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          bf16x4 tmp;
#pragma unroll
          for (int e = 0; e < 4; ++e) tmp[e] = static_cast<__bf16>(o[g][d][4 * r4 + e] * inv);
          *reinterpret_cast<u32x2 *>(op + d * 32 + r4 * 8) = __builtin_bit_cast(u32x2, tmp);
        }
    }
  }
}

// ------------------------------------------------------------------ bf16 kernel for few queries: keys split over the waves
// With fewer units of 128 queries than compute units (2300 tokens at four heads are 72) the kernel above leaves most of the chip
// idle and every wave walks all keys, 36 blocks of 64 one after the other: 41 us.  Here a work-group takes 32 queries and its four
// waves take every fourth block of 32 keys each, with a softmax of their own and without a barrier; the four meet once in LDS,
// added in wave order: 288 work-groups of 18 blocks, 22 us (642 tokens at four heads 13.9 and 7.9).  What bounds it is the path that
// feeds K and V from L2 (every 32 queries read all of them) and the chain of a wave's blocks; so it is for few queries only, see attention_plan.h.
//
// A wave's K and V tiles (32 keys, 4 KiB each) go through a ring of its own of five tiles in the order K0 V0 K1 V1 ...: when
// tile i has been read its place takes tile i + 5, so two blocks are in flight and two work-groups fit a compute unit.  Fragments and
// swizzles are those of the kernels above.  A reference is of a wave's keys and moves for all of its queries at once, and the row sums are a lane's own, so the
// last bits are not those of the kernels above; a wave whose first 32 keys all have logits of -inf for a query leaves that query not a number.
template <int DH, bool QS, bool ST>
__global__ __launch_bounds__(256, 2) void tiles_attention_split_bf16_kernel(AttnArgs a) {
  static_assert(DH == 64, "fragment tables below");
  constexpr int ROWB = DH * 2, TILE = 32 * ROWB, RING = 5, NKS = DH / 16;
  __shared__ __align__(1024) unsigned char smem[4 * RING * TILE];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int ld = 3 * a.D, ld2 = ld * 2;
  const int QB = a.QB * 4;                                       // units of 32 queries
  const int logical = xcd_remap_attn(blockIdx.x, a.total * 4);
  const int qb = logical % QB;
  int rest = logical / QB;
  const int head = rest % a.heads;
  rest /= a.heads;
  const int tile = rest % a.T, b = rest / a.T;
  const tile_desc &td = a.tiles[tile];
  const int n_t = td.n_tok, q0 = qb * 32;
  if (q0 >= n_t) return;                                         // uniform
  const int bw = td.X1 - td.X0;
  if constexpr (ST) {                                            // no query of these belongs to the tile
    const int lo = (td.y0 - td.Y0) * bw + (td.x0 - td.X0), up = (td.y1 - 1 - td.Y0) * bw + (td.x1 - 1 - td.X0);
    if (q0 > up || q0 + 31 < lo) return;
  }
  const size_t row0 = static_cast<size_t>(b) * a.n_h + td.tok_off;
  const bf16_t *base = static_cast<const bf16_t *>(a.qkv) + row0 * ld + head * DH;
  const int blocks = (n_t + 31) / 32, mine = (blocks - wave + 3) / 4;      // this wave's blocks: wave, wave + 4, ...
  unsigned char *const ring = smem + wave * RING * TILE;

  // ---- load side: 4 KiB = 4 loads of 8 rows
  auto swzK = [](int r) { return (r & 7) ^ ((r >> 3) & 1); };
  auto swzV = [](int r) { return (((r >> 1) & 1) << 2) | (((r >> 3) & 1) << 1); };
  int offK[4], offV[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 8 * i + (lane >> 3);
    offK[i] = r * ld2 + ((lane & 7) ^ swzK(r)) * 16;
    offV[i] = r * ld2 + ((lane & 7) ^ swzV(r)) * 16;
  }
  // tile i of this wave: K (even) or V (odd) of its block i / 2; rows past the end re-read the last one (finite, masked)
  auto issue = [&](int i) {
    const int k0 = (wave + 4 * (i >> 1)) * 32, lim = n_t - 1 - k0;
    const unsigned char *g = reinterpret_cast<const unsigned char *>(base + ((i & 1) + 1) * a.D + static_cast<size_t>(k0) * ld);
    unsigned char *dst = ring + (i % RING) * TILE;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int back = max(8 * j + (lane >> 3) - lim, 0) * ld2;
      attn_dl_load16(reinterpret_cast<const bf16_t *>(g + static_cast<uint32_t>(((i & 1) ? offV[j] : offK[j]) - back)), dst + j * 1024);
    }
  };
  const int tiles = 2 * mine;
  bf16x8 qf[NKS];
  {
    const bf16_t *qp = base + static_cast<size_t>(min(q0 + l32, n_t - 1)) * ld + hi * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8 *>(qp + ks * 16);
  }
  for (int i = 0; i < RING && i < tiles; ++i) issue(i);

  // ---- read side (see the kernel above)
  const int kr = key_perm(l32), k_row = kr * ROWB, k_swz = swzK(kr), L16 = lane & 15;
  unsigned v_addr[2][2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int vr = 8 * hi + 4 * e + (L16 >> 2);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const int o = 32 * d + 16 * ((lane >> 4) & 1) + 4 * (L16 & 3);
      v_addr[e][d] = vr * ROWB + (((o >> 3) ^ swzV(vr)) << 4) + ((o >> 2) & 1) * 8;
    }
  }
  // tile i has landed; with four or more tiles behind it their loads stay in flight
  auto landed = [&](int i) {
    if (i + RING <= tiles) __builtin_amdgcn_s_waitcnt(0x0F70 | (16 & 15) | ((16 >> 4) << 14));
    else __builtin_amdgcn_s_waitcnt(0x0F70);
    __builtin_amdgcn_sched_barrier(0);
  };
  f32x16 o[2], minit;
#pragma unroll
  for (int r = 0; r < 16; ++r) o[0][r] = o[1][r] = minit[r] = 0.f;
  float lsum = 0.f;
  const float c = QS ? 1.0f : a.scale_log2, TAU = 10.0f / c;
  bool have_ref = false;
  const unsigned ring0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)ring));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const bf16x2 one2 = {static_cast<__bf16>(1.0f), static_cast<__bf16>(1.0f)};
  for (int n = 0; n < mine; ++n) {
    landed(2 * n);
    const unsigned char *st = ring + (2 * n % RING) * TILE;
    bf16x8 kf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) kf[ks] = *reinterpret_cast<const bf16x8 *>(st + k_row + (((2 * ks + hi) ^ k_swz) << 4));
    f32x16 s;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[ks], qf[ks], ks == 0 ? minit : s, 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);      // the fragments are in registers: their place may be loaded again
    if (2 * n + RING < tiles) issue(2 * n + RING);
    const int k0 = (wave + 4 * n) * 32;
    if (k0 + 32 > n_t) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (k0 + 16 * (r / 8) + 8 * hi + (r % 8) >= n_t) s[r] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
    {
      unsigned m_lo, m_up;
      lane_pair_exchange(__builtin_bit_cast(unsigned, mx), m_lo, m_up);
      mx = fmaxf(__builtin_bit_cast(float, m_lo), __builtin_bit_cast(float, m_up));      // finite: every block holds a valid key
    }
    if (!have_ref || __any(mx > TAU)) {
      const float d = have_ref ? fmaxf(mx, 0.f) : mx;
      const float alpha = have_ref ? __builtin_amdgcn_exp2f(-d * c) : 0.f;
      const float ninit = minit[0] - d;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        s[r] -= d;
        o[0][r] *= alpha;
        o[1][r] *= alpha;
        minit[r] = ninit;
      }
      lsum *= alpha;
      have_ref = true;
    }
    bf16x8 pf[2];
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
      for (int e = 0; e < 8; ++e) pf[h2][e] = static_cast<__bf16>(__builtin_amdgcn_exp2f(QS ? s[8 * h2 + e] : s[8 * h2 + e] * c));
    landed(2 * n + 1);
    const unsigned vbase = ring0 + (2 * n + 1) % RING * TILE;
    unsigned va[2][2];
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int d = 0; d < 2; ++d) va[e][d] = vbase + v_addr[e][d];
    VFrag64 vf;
    v_frag_issue<0>(vf, va);
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
      for (int i = 0; i < 4; ++i) lsum = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{pf[h2][2 * i], pf[h2][2 * i + 1]}, one2, lsum, false);
    v_frag_wait(vf);
    __builtin_amdgcn_sched_barrier(0);
    if (2 * n + 1 + RING < tiles) issue(2 * n + 1 + RING);
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2)
#pragma unroll
      for (int d = 0; d < 2; ++d) {
        typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
        const u64x2 both = {vf.r[h2][d][0], vf.r[h2][d][1]};
        o[d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, both), pf[h2], o[d], 0, 0, 0);
      }
  }

  // ---- the four waves meet: references and sums first, then the outputs, each wave's part of the features
  __syncthreads();                                               // nobody reads or loads a ring any more
  float *const stat = reinterpret_cast<float *>(smem);           // [4][2][32]
  float *const box = stat + 4 * 2 * 32;                          // [4][32][64]
  {
    unsigned l_lo, l_up;
    lane_pair_exchange(__builtin_bit_cast(unsigned, lsum), l_lo, l_up);
    if (hi == 0) {
      stat[(wave * 2) * 32 + l32] = have_ref ? -minit[0] * c : -INFINITY;      // a wave without keys
      stat[(wave * 2 + 1) * 32 + l32] = __builtin_bit_cast(float, l_lo) + __builtin_bit_cast(float, l_up);
    }
  }
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) box[(wave * 32 + d * 16 + r) * 64 + lane] = o[d][r];
  __syncthreads();
  float top = stat[l32], f[4], total = 0.f;                      // wave 0 has the first block: finite
#pragma unroll
  for (int w = 1; w < 4; ++w) top = fmaxf(top, stat[w * 2 * 32 + l32]);
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    f[w] = __builtin_amdgcn_exp2f(stat[w * 2 * 32 + l32] - top);
    total = fmaf(stat[(w * 2 + 1) * 32 + l32], f[w], total);
  }
  const int qrow = q0 + l32;
  if (qrow >= n_t) return;
  size_t orow = row0 + qrow;
  if constexpr (ST) {
    const int yy = td.Y0 + qrow / bw, xx = td.X0 + qrow % bw;
    if (!(yy >= td.y0 && yy < td.y1 && xx >= td.x0 && xx < td.x1)) return;
    orow = static_cast<size_t>(b) * a.N + static_cast<size_t>(yy) * a.Wp + xx;
  }
  const float inv = 1.0f / total;
  if (!ST && a.lse && wave == 0 && hi == 0)
    a.lse[(static_cast<size_t>(b) * a.heads + head) * a.n_h + td.tok_off + qrow] = (__builtin_amdgcn_logf(total) + top) * 0.69314718055994531f;
  bf16_t *op = static_cast<bf16_t *>(a.out) + orow * a.D + head * DH + hi * 4 + (wave >> 1) * 32 + (wave & 1) * 16;
#pragma unroll
  for (int p = 0; p < 2; ++p) {                                  // registers 4 r4 .. + 3 of feature block wave / 2, r4 = 2 (wave % 2) + p
    bf16x4 tmp;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int r = (wave >> 1) * 16 + (wave & 1) * 8 + 4 * p + e;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) v = fmaf(box[(w * 32 + r) * 64 + lane], f[w], v);
      tmp[e] = static_cast<__bf16>(v * inv);
    }
    *reinterpret_cast<u32x2 *>(op + p * 8) = __builtin_bit_cast(u32x2, tmp);
  }
}

// ------------------------------------------------------------------ fp32 path
// 32 queries of one (sample, tile, head) per work-group, MFMA 32x32x2 in fp32 with operands straight from global memory.
// The four waves take every fourth block of 32 keys, each with a softmax of its own (running maximum, sum and output);
// the four are merged through LDS in wave order.  As in the bf16 kernel S^T = K Q^T is computed, so a lane owns a query
// column, and the accumulator registers of S^T are the B operand of O^T = V^T P^T: register 4 q + j of lane half hi
// holds key 8 q + 4 hi + j, so matrix step (q, j) multiplies keys 8 q + j and 8 q + 4 + j.  The tiny workload (128
// tokens a tile, head dimension 32) takes 5 us; one work-group per query with a reduction over LDS took 20.
// NB: 32-feature blocks of the output a work-group takes (wider heads: more work-groups, each with all the scores),
// VEC4: the head's rows start on 16 bytes.
template <int NB, bool VEC4>
__global__ __launch_bounds__(256) void tiles_attention_f32_kernel(AttnArgs a, int dh) {
  __shared__ float stat[4][2][32];
  __shared__ float box[4][16][64];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hi = lane >> 5;
  const int qb = blockIdx.x % a.QB, head = blockIdx.y, tile = (blockIdx.x / a.QB) % a.T, b = blockIdx.x / a.QB / a.T;
  const int n_t = a.tiles[tile].n_tok, q0 = qb * 32;
  if (q0 >= n_t) return;                                     // uniform
  const int64_t row0 = static_cast<int64_t>(b) * a.n_h + a.tiles[tile].tok_off;
  const int ld = 3 * a.D;
  const float *base = static_cast<const float *>(a.qkv) + row0 * ld + head * dh;
  auto quad = [&](const float *row, int k) {                 // row[k .. k + 3], zero past the head
    if constexpr (VEC4) {
      return k < dh ? *reinterpret_cast<const float4 *>(row + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
      return make_float4(k < dh ? row[k] : 0.f, k + 1 < dh ? row[k + 1] : 0.f, k + 2 < dh ? row[k + 2] : 0.f, k + 3 < dh ? row[k + 3] : 0.f);
    }
  };
  const float scale = rsqrtf(static_cast<float>(dh));
  const int steps = (dh + 7) / 8, f0 = blockIdx.z * NB * 32;      // output features of this work-group
  const float *qrow = base + static_cast<size_t>(min(q0 + l32, n_t - 1)) * ld;
  f32x16 o[NB] = {};
  float mx = -INFINITY, sum = 0.f;
  for (int k0 = wave * 32; k0 < n_t; k0 += 128) {
    const float *krow = base + a.D + static_cast<size_t>(min(k0 + l32, n_t - 1)) * ld;
    f32x16 s = {};
    for (int st = 0; st < steps; st += 4) {                  // of eight features, four at a time
      float4 kv[4], qv[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        kv[i] = quad(krow, 8 * (st + i) + 4 * hi);
        qv[i] = quad(qrow, 8 * (st + i) + 4 * hi);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[i].x, qv[i].x, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[i].y, qv[i].y, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[i].z, qv[i].z, s, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[i].w, qv[i].w, s, 0, 0, 0);
      }
    }
    // the values are requested ahead of the softmax
    float vv[NB][16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r / 4) + 4 * hi + r % 4;                     // past the tile: zero times zero
      const float *vrow = base + 2 * a.D + static_cast<size_t>(min(key, n_t - 1)) * ld;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int f = f0 + nb * 32 + l32;
        vv[nb][r] = f < dh && key < n_t ? vrow[f] : 0.f;
      }
    }
    float top = -INFINITY;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 8 * (r / 4) + 4 * hi + r % 4;
      s[r] = key < n_t ? s[r] * scale : -INFINITY;
      top = fmaxf(top, s[r]);
    }
    top = fmaxf(mx, fmaxf(top, __shfl_xor(top, 32)));
    const float ref = top == -INFINITY ? 0.f : top;          // every score so far overflowed to -inf: weights of zero
    const float alpha = expf(mx - ref);
    mx = top;
    float part = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      s[r] = expf(s[r] - ref);
      part += s[r];
    }
    sum = fmaf(sum, alpha, part);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[nb][r] *= alpha;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) o[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[nb][r], s[r], o[nb], 0, 0, 0);
  }
  sum += __shfl_xor(sum, 32);                                // the two halves hold different keys of the same query
  if (hi == 0) {
    stat[wave][0][l32] = mx;
    stat[wave][1][l32] = sum;
  }
  __syncthreads();
  float m_all = stat[0][0][l32], total = 0.f;
#pragma unroll
  for (int w = 1; w < 4; ++w) m_all = fmaxf(m_all, stat[w][0][l32]);
#pragma unroll
  for (int w = 0; w < 4; ++w) total += stat[w][1][l32] * expf(stat[w][0][l32] - m_all);      // a wave without keys: 0 * exp(-inf)
  const int qi = q0 + l32;
  if (a.lse && f0 == 0 && wave == 0 && hi == 0 && qi < n_t)
    a.lse[(static_cast<size_t>(b) * a.heads + head) * a.n_h + a.tiles[tile].tok_off + qi] = m_all + logf(total);
  const float f_own = expf(mx - m_all) / total;
  float *orow = static_cast<float *>(a.out) + (row0 + min(qi, n_t - 1)) * a.D + head * dh;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) box[wave][r][lane] = o[nb][r] * f_own;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {                            // wave w adds up registers 4 w .. 4 w + 3: features 8 w + 4 hi + j
      const int r = 4 * wave + j, f = f0 + nb * 32 + 8 * wave + 4 * hi + j;
      const float v = (box[0][r][lane] + box[1][r][lane]) + (box[2][r][lane] + box[3][r][lane]);
      if (qi < n_t && f < dh) orow[f] = v;
    }
  }
}

// at dh = 64, 0: what attention_plan.h names (default); 1: 128-key blocks, two work-groups per CU; 2: one query group a wave; 3, 4: two groups, work-groups of two, four waves
static int g_attn_variant = 0;
static int g_attn_cus = 0;

hipError_t attention_init() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  return hipDeviceGetAttribute(&g_attn_cus, hipDeviceAttributeMultiprocessorCount, dev);
}
bool attention_accepts_prescaled_q() { return true; }

SeqGeom ctx_geom(const reslim_ctx *c) {
  SeqGeom g;
  g.d_tiles = c->d_tiles;
  g.d_tile_of_tok = c->d_tile_of_tok;
  g.T = c->T;
  g.n_h = c->n_h;
  g.max_n_tok = c->max_n_tok;
  g.pairs = 0;
  g.pairs_owned = 0;
  g.blocks128 = g.blocks256 = 0;
  for (const tile_desc &t : c->tiles) {
    g.blocks128 += (t.n_tok + 127) / 128;
    g.blocks256 += (t.n_tok + 255) / 256;
    g.pairs += static_cast<double>(t.n_tok) * t.n_tok;
    g.pairs_owned += static_cast<double>(t.y1 - t.y0) * (t.x1 - t.x0) * t.n_tok;
  }
  return g;
}

// PQK, PPV: wave priority during the score and the P V matrix instructions
template <int DH, int BKV, int MINW, int PQK = 1, int PPV = 1>
static void launch_bf16_variant(const AttnArgs &a, bool q_prescaled, bool stitched, int grid, hipStream_t st) {
  if (stitched) {
    if (q_prescaled) tiles_attention_bf16_kernel<DH, BKV, true, MINW, true, PQK, PPV><<<dim3(grid), dim3(256), 0, st>>>(a);
    else tiles_attention_bf16_kernel<DH, BKV, false, MINW, true, PQK, PPV><<<dim3(grid), dim3(256), 0, st>>>(a);
  } else {
    if (q_prescaled) tiles_attention_bf16_kernel<DH, BKV, true, MINW, false, PQK, PPV><<<dim3(grid), dim3(256), 0, st>>>(a);
    else tiles_attention_bf16_kernel<DH, BKV, false, MINW, false, PQK, PPV><<<dim3(grid), dim3(256), 0, st>>>(a);
  }
}

template <int NW>
static void launch_pair(const AttnArgs &a, bool q_prescaled, bool stitched, hipStream_t st) {
  const dim3 grid(a.total), blk(64 * NW);
  if (stitched) {
    if (q_prescaled) tiles_attention_pair_bf16_kernel<true, true, NW><<<grid, blk, 0, st>>>(a);
    else tiles_attention_pair_bf16_kernel<false, true, NW><<<grid, blk, 0, st>>>(a);
  } else {
    if (q_prescaled) tiles_attention_pair_bf16_kernel<true, false, NW><<<grid, blk, 0, st>>>(a);
    else tiles_attention_pair_bf16_kernel<false, false, NW><<<grid, blk, 0, st>>>(a);
  }
}

hipError_t launch_tiles_attention(const reslim_ctx *c, const void *qkv, void *out, int batch, bool q_prescaled,
                                  hipStream_t st, float *lse, const SeqGeom *geom, bool stitched) {
  const SeqGeom own = geom ? *geom : ctx_geom(c);
  const SeqGeom &sg = own;
  AttnArgs a;
  a.qkv = qkv;
  a.out = out;
  a.lse = lse;
  a.tiles = sg.d_tiles;
  a.T = sg.T;
  a.heads = c->cfg.heads;
  a.D = c->cfg.embed_dim;
  a.n_h = sg.n_h;
  a.scale_log2 = 1.4426950408889634f / sqrtf(static_cast<float>(c->dh));
  a.Wp = 0;
  a.N = 0;
  if (stitched) {                          // the context's own tiling, bf16 kernel, no log-sum-exp rows
    if (geom || lse || c->cfg.dtype != RESLIM_BF16) return hipErrorInvalidValue;
    a.Wp = c->Wp;
    a.N = c->N;
  }
  if (c->cfg.dtype == RESLIM_BF16) {
    a.QB = (sg.max_n_tok + 127) / 128;
    const int64_t sets = static_cast<int64_t>(batch) * a.heads, total = sets * sg.T * a.QB;
    if (total > INT32_MAX) return hipErrorInvalidValue;
    a.total = static_cast<int>(total);
    if (a.total == 0) return hipSuccess;
    if (g_attn_cus <= 0) return hipErrorInvalidValue;
    const int pg2 = a.total < 2 * g_attn_cus ? a.total : 2 * g_attn_cus;   // persistent grids
    const int pg3 = a.total < 3 * g_attn_cus ? a.total : 3 * g_attn_cus;
    const int nw = c->dh != 64 ? 0 : g_attn_variant == 0 ? attn_pair_waves(sets * sg.blocks128, sets * sg.blocks256, g_attn_cus, sg.max_n_tok) : g_attn_variant == 3 ? 2 : g_attn_variant == 4 ? 4 : 0;
    const bool pair_fits = nw > 0 && sets * sg.T * ((sg.max_n_tok + 64 * nw - 1) / (64 * nw)) <= most_work_groups(64 * nw);
    if (c->dh == 64 && g_attn_variant == 0 && attn_split_keys(a.total, g_attn_cus, sg.max_n_tok)) {
      const dim3 grid(4 * a.total), blk(256);
      if (stitched && q_prescaled) tiles_attention_split_bf16_kernel<64, true, true><<<grid, blk, 0, st>>>(a);
      else if (stitched) tiles_attention_split_bf16_kernel<64, false, true><<<grid, blk, 0, st>>>(a);
      else if (q_prescaled) tiles_attention_split_bf16_kernel<64, true, false><<<grid, blk, 0, st>>>(a);
      else tiles_attention_split_bf16_kernel<64, false, false><<<grid, blk, 0, st>>>(a);
    } else if (pair_fits) {
      a.QB = (sg.max_n_tok + 64 * nw - 1) / (64 * nw);
      a.total = static_cast<int>(sets * sg.T * a.QB);
      if (nw == 2) launch_pair<2>(a, q_prescaled, stitched, st);
      else launch_pair<4>(a, q_prescaled, stitched, st);
    } else if (c->dh == 64 && g_attn_variant != 1) launch_bf16_variant<64, 64, 3, 2, 1>(a, q_prescaled, stitched, pg3, st);
    else if (c->dh == 64) launch_bf16_variant<64, 128, 2>(a, q_prescaled, stitched, pg2, st);
    else if (c->dh == 128) launch_bf16_variant<128, 64, 2>(a, q_prescaled, stitched, pg2, st);
    else if (c->dh == 256) {
      // 128 output-accumulator and 64 query-fragment registers per lane: one work-group per CU
      const int pg1 = a.total < g_attn_cus ? a.total : g_attn_cus;
      launch_bf16_variant<256, 32, 1>(a, q_prescaled, stitched, pg1, st);
    } else {
      return hipErrorInvalidValue;
    }
    return hipGetLastError();
  }
  a.QB = (sg.max_n_tok + 31) / 32;
  a.total = 0;
  const int64_t groups = static_cast<int64_t>(a.QB) * sg.T * batch;
  if (groups > INT32_MAX || a.heads > 65535) return hipErrorInvalidValue;
  const int nb = (c->dh + 31) / 32;
  const dim3 grid(static_cast<unsigned>(groups), a.heads, (nb + 7) / 8), blk(256);
  const bool vec = c->dh % 4 == 0 && a.D % 4 == 0 && (reinterpret_cast<uintptr_t>(qkv) & 15) == 0;
#define RESLIM_ATTN32(NB) (vec ? tiles_attention_f32_kernel<NB, true><<<grid, blk, 0, st>>>(a, c->dh) : tiles_attention_f32_kernel<NB, false><<<grid, blk, 0, st>>>(a, c->dh))
  if (nb <= 1) RESLIM_ATTN32(1);
  else if (nb <= 2) RESLIM_ATTN32(2);
  else if (nb <= 4) RESLIM_ATTN32(4);
  else RESLIM_ATTN32(8);
#undef RESLIM_ATTN32
  return hipGetLastError();
}

}  // namespace reslim

// tuning hook for dh = 64: 0 = the kernel that attention_plan.h names (default), 1 = 128-key blocks, one query group a wave, two work-groups per CU, 2 = 64-key
// blocks, one query group a wave, 3 and 4 = two query groups a wave, two and four waves to a work-group
extern "C" void reslim_debug_set_attention_variant(int v) { reslim::g_attn_variant = v; }
