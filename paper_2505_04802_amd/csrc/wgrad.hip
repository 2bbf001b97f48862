// Weight gradient of a linear layer y = x W^T + b (training of the model of ORBIT-2
// Sec. 4.1; the chain rule gives  dW[n][k] = sum_m dY[m][n] * X[m][k]  and  db[n] = sum_m dY[m][n]):
// a contraction over the TOKENS, the leading index of both operands, so neither is "k-contiguous"
// the way the forward GEMM wants them.  Instead of transposing activations in HBM the kernel reads
// both operands as they lie, [token][feature] row-major, straight into LDS, and fetches both MFMA
// operands with the TRANSPOSING LDS read ds_read_b64_tr_b16: a lane gets 8 consecutive tokens of one
// feature column, which is exactly the k-slice of an A operand (feature = output row n, from dY) or
// a B operand (feature = k, from X).
//
// A work-group owns a tile of dW for a slice of the tokens (dW is small and M is huge); fp32 partial
// tiles are summed in a fixed order afterwards (deterministic, no atomics).  The four products of a
// block run as ONE launch over a common tile list with common slices: at D = 256 and 19,552 tokens
// they took 104 us one by one plus 110 us for the bias sums, most of it partial tiles (64 slices of
// every product, 192 MB a block) and start-up; together 45 us (10 slices, 31 MB), bias sums included.  At D = 1024 and 161,408 tokens (c2) the four products took 4.00 ms and
// the bias sums 0.56; the two launches of such a block take 2.40 + 1.19 ms, 1130 TFLOP/s, with the matrix pipe busy 88 % of
// the cycles of a clock of 1.2 GHz (1600 TFLOP/s on operands of zeros): the chip's power limit.
#include <type_traits>

#include "attention_common.h"

namespace reslim {

// One launch takes up to four products of the same number of tokens (the linear layers of a block), each with its own
// list of tiles; the token slices are common to all.
struct WgradArgs {
  const bf16_t *dy[kWgradMax];      // [M, N]
  const bf16_t *x[kWgradMax];       // [M, K]
  float *out[kWgradMax];            // per token slice a partial [N, K] (one slice: the gradient itself)
  float *out_b[kWgradMax];          // likewise: the column sums of dY, [N]
  int N[kWgradMax], K[kWgradMax];
  int tiles_n[kWgradMax], tiles_k[kWgradMax];
  int end[kWgradMax];               // one past the last tile of this product in the common list
  int M, tiles;
  int m_per_split;       // tokens per slice, a multiple of 64
  int64_t split_stride;  // floats between the slices of out and of out_b
};

// Product and tile of this work-group.  The arguments of all products are read at once and selected from: a chain of
// loads, each with an address that depends on the one before, costs microseconds at the start of every launch (arguments
// lie in host memory).  Column strips of 8 tiles, row-major inside a strip: consecutive tiles share operands.
struct WgradTile {
  const bf16_t *dy, *x;
  float *out, *out_b;
  int N, K, tn, tk, split;
  __device__ __forceinline__ WgradTile(const WgradArgs &a, int slot) {
    constexpr int SW = 8;
    split = __builtin_amdgcn_readfirstlane(slot / a.tiles);      // divisions run on the vector units
    int L = slot - split * a.tiles;
    const int e0 = a.end[0], e1 = a.end[1], e2 = a.end[2];
    const bool i1 = L >= e0, i2 = L >= e1, i3 = L >= e2;
    static_assert(kWgradMax == 4, "selection below");
    auto pick = [&](auto v0, auto v1, auto v2, auto v3) { return i3 ? v3 : i2 ? v2 : i1 ? v1 : v0; };
    dy = pick(a.dy[0], a.dy[1], a.dy[2], a.dy[3]);
    x = pick(a.x[0], a.x[1], a.x[2], a.x[3]);
    out = pick(a.out[0], a.out[1], a.out[2], a.out[3]);
    out_b = pick(a.out_b[0], a.out_b[1], a.out_b[2], a.out_b[3]);
    N = pick(a.N[0], a.N[1], a.N[2], a.N[3]);
    K = pick(a.K[0], a.K[1], a.K[2], a.K[3]);
    const int tiles_n = pick(a.tiles_n[0], a.tiles_n[1], a.tiles_n[2], a.tiles_n[3]);
    const int tiles_k = pick(a.tiles_k[0], a.tiles_k[1], a.tiles_k[2], a.tiles_k[3]);
    L -= pick(0, e0, e1, e2);
    const int strip = L / (SW * tiles_n);
    const int wdt = min(SW, tiles_k - strip * SW);
    const int r = L - strip * SW * tiles_n;
    tn = __builtin_amdgcn_readfirstlane(r / wdt);
    tk = __builtin_amdgcn_readfirstlane(strip * SW + r % wdt);
  }
};

// Tiles of 128 RB x 256, two groups of waves taking turns.
//
// The schedule of the persistent GEMM (gemm_pp.inc) on operands whose contraction index is the ROW: a slab is 64 tokens
// of 128 RB columns of dY and 256 columns of X, in two LDS buffers; the two groups of four waves run half a phase apart,
// one reading fragments and issuing loads while the other has the matrix cores.  A phase multiplies one half of a wave's
// dW rows by both halves of its columns, 8 RB matrix instructions; the loads run up to 1.5 slabs ahead, with waits that
// count (the order of reuse is the one described there: phase 0 of slab s loads column half 0 of slab s + 2 and row half 1
// of slab s + 1, phase 1 row half 0 and column half 1 of slab s + 2).
//
// The unit of loading and reuse is a half tile: 64 tokens x 128 columns (64 for the rows at RB = 1), stored as rows of
// 256 (128) bytes.  A wave owns 32 RB rows of dW in either row half and 32 columns in either column half, so a half tile is
// a contiguous piece of the rows in memory (whole 128-byte lines).  Fragments come from the transposing read
// ds_read_b64_tr_b16; its 32 lanes touch 4 tokens x 64 bytes per LDS cycle, so the 16-byte chunks of rows 4r .. 4r + 3
// are moved to different banks (chunk ^= 4 (r & 3) + ((r >> 2) & 3) at 256-byte rows, 4 ((r >> 1) & 1) at 128-byte rows).
//
// Rows past the end of the slice lie beyond the buffer and are loaded as zeros; they add nothing.  Columns past the end
// of a matrix hold other columns' numbers (or zeros) and only reach outputs that are not stored.
//
// Bias gradient: the column sums of dY.  The fragments of dY are in registers anyway; in the work-groups of the first
// column tile each wave of a group adds up the tokens of one quarter of its slab on the vector units while the matrix
// cores run, which saves the pass over dY that the sums would take.

template <int OFF>
__device__ __forceinline__ void tr_read(uint64_t &d, unsigned addr) {
  static_assert(OFF >= 0 && OFF < 65536, "16-bit offset field");
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF) : "memory");
}
// sum of the four bfloat16 of a 64-bit fragment half
__device__ __forceinline__ float sum4_bf16(uint64_t v) {
  const uint32_t a = static_cast<uint32_t>(v), b = static_cast<uint32_t>(v >> 32);
  return (__uint_as_float(a << 16) + __uint_as_float(a & 0xffff0000u)) + (__uint_as_float(b << 16) + __uint_as_float(b & 0xffff0000u));
}
template <int N>
__device__ __forceinline__ void wgrad_wait_vm_lgkm0() {
  static_assert(N >= 0 && N < 64, "vmcnt field is 6 bits on gfx9");
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | ((N >> 4) << 14));
}

template <int RB>
__global__ __launch_bounds__(512, 2) void wgrad_bf16_kernel(WgradArgs a) {
  constexpr int TN = 128 * RB, TK = 256, BM = 64;
  constexpr int kRowN = 128 * RB, kRowK = 256;                         // bytes of a half-tile row in LDS
  constexpr int kHalfN = BM * kRowN, kHalfK = BM * kRowK;              // bytes of a half tile
  constexpr int kKBase = 4 * kHalfN;                                   // LDS: dY buffers 0, 1, then X buffers 0, 1
  constexpr int kPhaseLoads = 2 + RB;
  extern __shared__ __align__(1024) unsigned char smem[];

  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  const int hi = lane >> 5, l32 = lane & 31, L16 = lane & 15;
  // work-groups of one XCD take consecutive tiles of the same token slices, which share their operands through its L2
  const int nwg = gridDim.x;
  const int slot = (nwg % 8 == 0) ? (blockIdx.x % 8) * (nwg / 8) + blockIdx.x / 8 : blockIdx.x;
  const WgradTile op(a, slot);
  const int split = op.split, tn = op.tn, tk = op.tk;
  const int n0 = tn * TN, k0 = tk * TK;
  const int m_begin = split * a.m_per_split;
  const int m_end = min(a.M, m_begin + a.m_per_split);
  const int nblk = (m_end - m_begin + BM - 1) / BM;

  // ---- load side: half tiles are 1 KiB blocks of 4 (8) rows, two per wave (one)
  constexpr unsigned kRsrcFlags = 0x00020000;        // raw buffer, 32-bit data format
  const unsigned N2 = static_cast<unsigned>(op.N) * 2, K2 = static_cast<unsigned>(op.K) * 2;
  unsigned vo_n[RB], vo_k[2];
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    if constexpr (RB == 2) {
      const int ch = (lane & 15) ^ (((lane >> 4) << 2) | (wave & 3));
      vo_n[b] = (4 * (wave + 8 * b) + (lane >> 4)) * N2 + ch * 16;
    } else {
      const int row = 8 * wave + (lane >> 3);
      vo_n[b] = row * N2 + (((lane & 7) ^ (((row >> 1) & 1) << 2)) << 4);
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int ch = (lane & 15) ^ (((lane >> 4) << 2) | (wave & 3));
    vo_k[b] = (4 * (wave + 8 * b) + (lane >> 4)) * K2 + ch * 16;
  }
  const bf16_t *n_ptr = op.dy + static_cast<size_t>(m_begin) * op.N + n0;
  const bf16_t *k_ptr = op.x + static_cast<size_t>(m_begin) * op.K + k0;
  int rows_left = m_end - m_begin;
  __amdgpu_buffer_rsrc_t n_rsrc, k_rsrc;
  // the buffers hold exactly the rows of one slab that exist, from the tile's first column on
  auto set_slab = [&]() {
    const int rows = __builtin_amdgcn_readfirstlane(rows_left < 0 ? 0 : min(rows_left, BM));      // the clamp would make it a vector
    n_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(n_ptr), 0, rows ? rows * static_cast<int>(N2) - n0 * 2 : 0, kRsrcFlags);
    k_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(k_ptr), 0, rows ? rows * static_cast<int>(K2) - k0 * 2 : 0, kRsrcFlags);
  };
  auto next_slab = [&]() {
    rows_left -= BM;
    n_ptr += static_cast<size_t>(BM) * op.N;
    k_ptr += static_cast<size_t>(BM) * op.K;
    set_slab();
  };
  // the column of a half goes into the lane's offset: as a scalar offset it could exceed the size of an empty buffer,
  // and the hardware subtracts it from the size before it compares
  auto load1 = [&](__amdgpu_buffer_rsrc_t r, int lds, unsigned vo) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(smem + lds), 16, static_cast<int>(vo), 0, 0, 0);
  };
  auto issue_n = [&](int h, int buf) {
#pragma unroll
    for (int b = 0; b < RB; ++b) load1(n_rsrc, (2 * buf + h) * kHalfN + (wave + 8 * b) * 1024, vo_n[b] + h * kRowN);
  };
  auto issue_k = [&](int h, int buf) {
#pragma unroll
    for (int b = 0; b < 2; ++b) load1(k_rsrc, kKBase + (2 * buf + h) * kHalfK + (wave + 8 * b) * 1024, vo_k[b] + h * kRowK);
  };

  // ---- read side: this lane points at token row 8 hi + 4 e + (lane % 16) / 4 of a 16-token step and at the 4 columns
  // 16 ((lane / 16) & 1) + 4 (lane % 4) .. + 3 of a block of 32; steps, halves and buffers go into the offset field
  const unsigned lds0 = static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const unsigned char *)smem));
  unsigned n_at[2][RB], k_at[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int vr = 8 * hi + 4 * e + (L16 >> 2);
    const int fo = 16 * ((lane >> 4) & 1) + 4 * (L16 & 3);
    const int s256 = ((vr & 3) << 2) | ((vr >> 2) & 3), s128 = ((vr >> 1) & 1) << 2;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
      const int o = 32 * (wm * RB + i) + fo;
      n_at[e][i] = lds0 + vr * kRowN + (((o >> 3) ^ (RB == 2 ? s256 : s128)) << 4) + ((o >> 2) & 1) * 8;
    }
    const int o = 32 * wn + fo;
    k_at[e] = lds0 + kKBase + vr * kRowK + (((o >> 3) ^ s256) << 4) + ((o >> 2) & 1) * 8;
  }
  struct Frag { uint64_t r[4][2]; };         // [16-token step][e]
  Frag nf[RB], w0, w1, wnext;
  auto read_n = [&](auto buf, auto half) {
    constexpr int O = (2 * decltype(buf)::value + decltype(half)::value) * kHalfN;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        tr_read<O>(nf[i].r[0][e], n_at[e][i]);
        tr_read<O + 16 * kRowN>(nf[i].r[1][e], n_at[e][i]);
        tr_read<O + 32 * kRowN>(nf[i].r[2][e], n_at[e][i]);
        tr_read<O + 48 * kRowN>(nf[i].r[3][e], n_at[e][i]);
      }
  };
  auto read_k = [&](auto buf, auto half, Frag &f) {
    constexpr int O = (2 * decltype(buf)::value + decltype(half)::value) * kHalfK;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      tr_read<O>(f.r[0][e], k_at[e]);
      tr_read<O + 16 * kRowK>(f.r[1][e], k_at[e]);
      tr_read<O + 32 * kRowK>(f.r[2][e], k_at[e]);
      tr_read<O + 48 * kRowK>(f.r[3][e], k_at[e]);
    }
  };
  // the reads are complete from here on: nothing that uses them may move above
  auto landed = [&](Frag &f) {
    asm volatile("" : "+v"(f.r[0][0]), "+v"(f.r[0][1]), "+v"(f.r[1][0]), "+v"(f.r[1][1]), "+v"(f.r[2][0]), "+v"(f.r[2][1]),
                      "+v"(f.r[3][0]), "+v"(f.r[3][1]));
  };
  auto frag = [](const Frag &f, int s) {
    typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
    const u64x2 v = {f.r[s][0], f.r[s][1]};
    return __builtin_bit_cast(bf16x8, v);
  };

  f32x16 acc[2 * RB][2];                     // [row block: RB of half 0, RB of half 1][column half]
#pragma unroll
  for (int i = 0; i < 2 * RB; ++i)
#pragma unroll
    for (int w = 0; w < 2; ++w)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][w][r] = 0.f;
  float bsum[2 * RB];
#pragma unroll
  for (int i = 0; i < 2 * RB; ++i) bsum[i] = 0.f;
  const bool bias = op.out_b && tk == 0;

  auto multiply = [&](int nh, int kh, const Frag &f) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < RB; ++i)
        acc[RB * nh + i][kh] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag(nf[i], s), frag(f, s), acc[RB * nh + i][kh], 0, 0, 0);
  };
  auto add_bias = [&](int nh) {              // this wave's quarter of the tokens: step wn
    if (bias) {
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        uint64_t v0 = nf[i].r[0][0], v1 = nf[i].r[0][1];
#pragma unroll
        for (int s = 1; s < 4; ++s) {
          const uint64_t c0 = nf[i].r[s][0], c1 = nf[i].r[s][1];
          v0 = wn == s ? +c0 : +v0;
          v1 = wn == s ? +c1 : +v1;
        }
        bsum[RB * nh + i] += sum4_bf16(v0) + sum4_bf16(v1);
      }
    }
  };
  auto half_barrier = [&]() {                // bare: __syncthreads() would wait for every load
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto end_memory_half = [&](Frag &f) {
    __builtin_amdgcn_sched_barrier(0);
    wgrad_wait_vm_lgkm0<2 * kPhaseLoads>();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RB; ++i) landed(nf[i]);
    landed(f);
    half_barrier();
    __builtin_amdgcn_s_setprio(1);
  };
  auto end_matrix_half = [&]() {
    __builtin_amdgcn_s_setprio(0);
    half_barrier();
  };
  typedef std::integral_constant<int, 0> I0;
  typedef std::integral_constant<int, 1> I1;
  // one slab out of buffer B; w0 holds column half 0 on entry and the next slab's on exit
  auto slab = [&](auto b, auto o) {
    constexpr int B = decltype(b)::value, O = decltype(o)::value;
    read_n(b, I0{});
    read_k(b, I1{}, w1);
    issue_n(1, O);
    next_slab();
    issue_k(0, B);
    end_memory_half(w1);
    multiply(0, 0, w0);
    add_bias(0);
    multiply(0, 1, w1);
    end_matrix_half();
    read_n(b, I1{});
    read_k(o, I0{}, wnext);
    issue_n(0, B);
    issue_k(1, B);
    end_memory_half(wnext);
    multiply(1, 0, w0);
    add_bias(1);
    w0 = wnext;
    multiply(1, 1, w1);
    end_matrix_half();
  };

  // prologue: two slabs but for the second one's row half 1, the first column half into registers
  set_slab();
  issue_k(0, 0);
  issue_n(0, 0);
  issue_k(1, 0);
  issue_n(1, 0);
  next_slab();
  issue_k(0, 1);
  issue_n(0, 1);
  issue_k(1, 1);
  __builtin_amdgcn_sched_barrier(0);
  wgrad_wait_vm_lgkm0<0>();
  half_barrier();
  read_k(I0{}, I0{}, w0);
  __builtin_amdgcn_sched_barrier(0);
  wgrad_wait_vm_lgkm0<63>();
  __builtin_amdgcn_sched_barrier(0);
  landed(w0);
  half_barrier();                            // both groups hold their first column half: its place may be loaded again
  if (wm == 1) half_barrier();               // from here on the second group is half a phase behind
  for (int g = 0; g < nblk; g += 2) {
    slab(I0{}, I1{});
    if (g + 1 < nblk) slab(I1{}, I0{});
  }
  if (wm == 0) half_barrier();               // the second group's last half
  wgrad_wait_vm_lgkm0<0>();                  // loads past the last slab still name this work-group's LDS

  // ---- store: accumulator register r of lane (l32, hi) is row 8 (r / 4) + 4 hi + r % 4, column l32
  auto store = [&](auto edge) {
    float *out = op.out + static_cast<size_t>(split) * a.split_stride + static_cast<size_t>(n0) * op.K + k0;
#pragma unroll
    for (int nh = 0; nh < 2; ++nh)
#pragma unroll
      for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int n = nh * 64 * RB + (wm * RB + i) * 32 + 8 * (r / 4) + 4 * hi + (r % 4);
          float *row = out + static_cast<size_t>(n) * op.K + wn * 32 + l32;
#pragma unroll
          for (int kh = 0; kh < 2; ++kh)
            if (!decltype(edge)::value || (n0 + n < op.N && k0 + kh * 128 + wn * 32 + l32 < op.K)) row[kh * 128] = acc[RB * nh + i][kh][r];
        }
  };
  if (n0 + TN <= op.N && k0 + TK <= op.K) store(std::integral_constant<bool, false>{});
  else store(std::integral_constant<bool, true>{});
  if (bias) {                                // uniform: the eight waves' quarters are added in a fixed order
    float *sm = reinterpret_cast<float *>(smem);      // [4][TN]
    __syncthreads();
#pragma unroll
    for (int nh = 0; nh < 2; ++nh)
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        const float v = bsum[RB * nh + i] + __shfl_xor(bsum[RB * nh + i], 32);
        if (hi == 0) sm[wn * TN + nh * 64 * RB + (wm * RB + i) * 32 + l32] = v;
      }
    __syncthreads();
    float *ob = op.out_b + static_cast<size_t>(split) * a.split_stride;
    if (t < TN && n0 + t < op.N) ob[n0 + t] = (sm[t] + sm[TN + t]) + (sm[2 * TN + t] + sm[3 * TN + t]);
  }
}

// fp32 path: one thread per element of dW
__global__ __launch_bounds__(256) void wgrad_f32_kernel(const float *__restrict__ dy, const float *__restrict__ x,
                                                        float *__restrict__ out, int M, int N, int K) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (idx >= static_cast<int64_t>(N) * K) return;
  const int n = static_cast<int>(idx / K), k = static_cast<int>(idx % K);
  float acc = 0.f;
  for (int m = 0; m < M; ++m) acc = fmaf(dy[static_cast<size_t>(m) * N + n], x[static_cast<size_t>(m) * K + k], acc);
  out[idx] = acc;
}

static int g_wgrad_cus = 256;
template <int RB>
constexpr int wgrad_lds() { return 2 * 64 * 2 * (128 * RB + 256); }
hipError_t wgrad_init() {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e == hipSuccess) e = hipDeviceGetAttribute(&g_wgrad_cus, hipDeviceAttributeMultiprocessorCount, dev);
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad_bf16_kernel<1>), hipFuncAttributeMaxDynamicSharedMemorySize, wgrad_lds<1>());
  if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void *>(&wgrad_bf16_kernel<2>), hipFuncAttributeMaxDynamicSharedMemorySize, wgrad_lds<2>());
  return e;
}

static WgradPlan wgrad_plan(const WgradOp *op, int n_op, int M) { return wgrad_plan(op, n_op, M, g_wgrad_cus); }

// Sum of the slices in a fixed order, to where the gradients belong.  A thread owns four adjacent numbers (every piece is
// a multiple of 8 long) of every G-th slice, with up to eight 16-byte loads in flight; the G groups are added through LDS.
struct WgradReduceArgs {
  const float4 *partial;
  int64_t stride4, end4[2 * kWgradMax];
  float *out[2 * kWgradMax];
  int n_part;
};
template <int G>
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(WgradReduceArgs a) {
  constexpr int COLS = 256 / G;
  __shared__ float4 sm[G > 1 ? 256 : 1];
  const int col = threadIdx.x % COLS, grp = threadIdx.x / COLS;
  const int64_t j = static_cast<int64_t>(blockIdx.x) * COLS + col;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  if (j < a.stride4) {
    int p = grp;
    for (; p + 7 * G < a.n_part; p += 8 * G) {
      float4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = a.partial[(p + i * G) * a.stride4 + j];
#pragma unroll
      for (int i = 0; i < 8; ++i) { acc.x += v[i].x; acc.y += v[i].y; acc.z += v[i].z; acc.w += v[i].w; }
    }
    for (; p < a.n_part; p += G) {
      const float4 v = a.partial[p * a.stride4 + j];
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
  }
  if constexpr (G > 1) {
    sm[threadIdx.x] = acc;
    __syncthreads();
    if (grp > 0) return;
#pragma unroll
    for (int g = 1; g < G; ++g) {
      const float4 v = sm[g * COLS + col];
      acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
  }
  if (j >= a.stride4) return;
  int64_t begin = 0;
  float *out = a.out[0];
#pragma unroll
  for (int i = 1; i < 2 * kWgradMax; ++i) {
    const bool in = j >= a.end4[i - 1];
    begin = in ? +a.end4[i - 1] : +begin;
    out = in ? +a.out[i] : +out;
  }
  out += 4 * (j - begin);
  if ((reinterpret_cast<uintptr_t>(out) & 15) == 0) *reinterpret_cast<float4 *>(out) = acc;
  else { out[0] = acc.x; out[1] = acc.y; out[2] = acc.z; out[3] = acc.w; }
}

// bytes of scratch the gradients of these layers need (0: none)
size_t wgrad_ws_bytes(int dtype, const WgradOp *op, int n_op, int M) {
  if (dtype != RESLIM_BF16) {
    int n = 0;
    for (int i = 0; i < n_op; ++i) n = op[i].N > n ? op[i].N : n;
    return align256(static_cast<size_t>(colsum_slabs(M)) * n * sizeof(float));
  }
  const WgradPlan p = wgrad_plan(op, n_op, M);
  return p.splits > 1 ? align256(static_cast<size_t>(p.splits) * wgrad_slice(op, n_op) * sizeof(float)) : 0;
}

static hipError_t launch_wgrad_bf16(const WgradPlan &p, const WgradOp *op, int n_op, int M, void *ws, hipStream_t st) {
  if (p.splits > 1 && !ws) return hipErrorInvalidValue;
  WgradArgs a = {};
  WgradReduceArgs r = {};
  for (int i = 0; i < kWgradMax; ++i) a.end[i] = INT32_MAX;
  for (int i = 0; i < 2 * kWgradMax; ++i) r.end4[i] = INT64_MAX;
  float *part = static_cast<float *>(ws);
  int tiles = 0;
  int64_t at = 0;
  for (int i = 0; i < n_op; ++i) {
    const int64_t n_w = static_cast<int64_t>(op[i].N) * op[i].K;
    a.dy[i] = static_cast<const bf16_t *>(op[i].dy);
    a.x[i] = static_cast<const bf16_t *>(op[i].x);
    a.out[i] = p.splits > 1 ? part + at : op[i].dw;
    a.out_b[i] = p.splits > 1 ? part + at + n_w : op[i].db;
    a.N[i] = op[i].N;
    a.K[i] = op[i].K;
    a.tiles_n[i] = wgrad_tiles_n(p.kind, a.N[i]);
    a.tiles_k[i] = (op[i].K + 255) / 256;
    a.end[i] = tiles += a.tiles_n[i] * a.tiles_k[i];
    r.out[2 * i] = op[i].dw;
    r.out[2 * i + 1] = op[i].db;
    r.end4[2 * i] = (at + n_w) / 4;
    at += n_w + a.N[i];
    r.end4[2 * i + 1] = at / 4;
  }
  a.split_stride = at;
  a.M = M;
  a.tiles = tiles;
  a.m_per_split = p.m_per_split;
  const dim3 grid(tiles * p.splits);
  if (p.kind == kWgrad256) wgrad_bf16_kernel<2><<<grid, dim3(512), wgrad_lds<2>(), st>>>(a);
  else wgrad_bf16_kernel<1><<<grid, dim3(512), wgrad_lds<1>(), st>>>(a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.splits == 1) return e;
  r.partial = static_cast<const float4 *>(ws);
  r.stride4 = at / 4;
  r.n_part = p.splits;
  // small gradients have many slices: four groups of threads share them, or too few loads are in flight
  if (p.splits >= 16) wgrad_reduce_kernel<4><<<dim3(static_cast<unsigned>((r.stride4 + 63) / 64)), dim3(256), 0, st>>>(r);
  else wgrad_reduce_kernel<1><<<dim3(static_cast<unsigned>((r.stride4 + 255) / 256)), dim3(256), 0, st>>>(r);
  return hipGetLastError();
}

// for each layer dW[N, K] = dY[M, N]^T X[M, K] and db[N] = column sums of dY, both fp32; ws as sized by wgrad_ws_bytes
hipError_t launch_wgrad(int dtype, const WgradOp *op, int n_op, int M, void *ws, hipStream_t st) {
  if (M <= 0 || n_op < 1 || n_op > kWgradMax) return hipErrorInvalidValue;
  for (int i = 0; i < n_op; ++i) {
    if (op[i].N <= 0 || op[i].K <= 0) return hipErrorInvalidValue;
    if (dtype == RESLIM_BF16 && (op[i].N % 8 != 0 || op[i].K % 8 != 0)) return hipErrorInvalidValue;
  }
  if (dtype == RESLIM_BF16) return launch_wgrad_bf16(wgrad_plan(op, n_op, M), op, n_op, M, ws, st);
  for (int i = 0; i < n_op; ++i) {
    const int64_t n = static_cast<int64_t>(op[i].N) * op[i].K;
    wgrad_f32_kernel<<<dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st>>>(
        static_cast<const float *>(op[i].dy), static_cast<const float *>(op[i].x), op[i].dw, M, op[i].N, op[i].K);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = launch_colsum(static_cast<const float *>(op[i].dy), static_cast<float *>(ws), op[i].db, M, op[i].N, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace reslim
