// Gradients of the whole model for one training step (ORBIT-2 Sec. 4.1 architecture and Bayesian
// training loss, Sec. 4.2 tiling, Sec. 5: the model is trained; Sec. 4.4: bf16 with gradient
// scaling).  The paper prints no gradient formula: everything here is the chain rule through the
// forward operations, walked backwards.  The blocks' gradient lives in backward.hip; this file
// holds the two ends of the model and the chaining:
//   loss            d_y = S (2 D (y - t) / n + 2 lambda / n sum_j b_ij sign(y_i - y_j)),  sign(0) = 0
//   back end        un-patchify transposed, head GEMM (input / weight / bias gradient), residual
//                   path (gradient of the 3x3 convolution's weights and bias), final LayerNorm on
//                   the interior tokens, zero gradient for the halo rows (their outputs are dropped)
//   front end       gather transposed (a patch adds up the gradients of its halo copies), position
//                   and resolution rows, output map of the aggregation, and the folded
//                   tokenisation + aggregation: gradients of the folded tables first (sums over
//                   tokens), then the chain rule through the fold to the unfolded parameters
// Mixed precision as in the block gradient: gradients that feed a GEMM are rounded to the
// activation type, sums are fp32, parameter gradients are fp32 and WRITTEN in a fixed summation
// order (deterministic).
#include <type_traits>
#include <algorithm>
#include <cmath>
#include <string>
#include <vector>

#include "common.h"

namespace reslim {

hipError_t launch_partial_reduce(const float *partial, float *out, int n_part, int64_t stride, int64_t n, hipStream_t st);

// ------------------------------------------------------------------ loss gradient
// Bound by memory: prediction and target read once, the gradient written once.  A thread owns four neighbouring columns and
// walks down RB rows with the three rows it needs in registers, so a pixel costs a quarter of a 16-byte load and half a
// 4-byte load of the prediction instead of nine 4-byte loads.  Rows of any length and alignment: the 16-byte accesses are
// of a type aligned to 4 bytes, which the hardware takes as they are; only the thread at a ragged row's end goes column by
// column (EVEN: there is none; its branches cost 4 % at 16 planes of 512 x 1024).  One thread per pixel took 9.2 ms at c3
// where this takes 2.5; loss and gradient of 32 planes of 1024 x 2050 took 818 us with ragged rows left to one thread
// per pixel, and take 297.
// The gradient is stored past the caches: it is as large as what the caches should keep of the two inputs, and what that buys is that
// inputs stay there until they are used again: 4 x 8 planes of 512 x 1024, value and gradient on a few sets of inputs in
// turn, 67.2 -> 62.8 us.  On inputs that lie in no cache it gains nothing to speak of (92 -> 89 us with the value's last kernel, which
// became faster too).  One plane set of 16 x 5760 x 11520 2.48 -> 2.42 ms.
// A neighbour outside the plane is held as NaN: every comparison with it is false, so its sign term is zero, which is
// what leaving it out means.  The sums of signs are small integers, exact in any order.
template <int RB, bool EVEN>
__global__ __launch_bounds__(256) void bayes_loss_bwd_kernel(const float *__restrict__ pred, const float *__restrict__ target,
                                                             const float *__restrict__ lat_w, float *__restrict__ d_pred,
                                                             int Hf, int Wf, float data_f, float tv_f) {
  const int64_t first = (static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x) * 4;
  if (first >= Wf) return;
  const int c0 = static_cast<int>(first), left = Wf - c0;      // columns from this thread's first to the row's end
  const size_t plane = static_cast<size_t>(blockIdx.z) * Hf * Wf;
  const float *xp = pred + plane;
  const int r_begin = blockIdx.y * RB, r_end = min(Hf, r_begin + RB);
  const float out_of_plane = __builtin_nanf("");
  auto sgn = [](float v) { return static_cast<float>((v > 0.f) - (v < 0.f)); };
  auto load4 = [&](const float *p, float (&v)[4]) {
    if (EVEN || left >= 4) {
      const float4_any m = *reinterpret_cast<const float4_any *>(p);
      v[0] = m.x; v[1] = m.y; v[2] = m.z; v[3] = m.w;
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = k < left ? p[k] : out_of_plane;
    }
  };
  auto load_row = [&](int r, float (&v)[6]) {      // columns c0 - 1 .. c0 + 4 of row r
    if (r < 0 || r >= Hf) {
#pragma unroll
      for (int k = 0; k < 6; ++k) v[k] = out_of_plane;
      return;
    }
    const float *row = xp + static_cast<size_t>(r) * Wf + c0;
    float m[4];
    load4(row, m);
    v[0] = c0 > 0 ? row[-1] : out_of_plane;
    v[1] = m[0]; v[2] = m[1]; v[3] = m[2]; v[4] = m[3];
    v[5] = left > 4 ? row[4] : out_of_plane;
  };
  float up[6], mid[6], dn[6];
  load_row(r_begin - 1, up);
  load_row(r_begin, mid);
#pragma unroll
  for (int i = 0; i < RB; ++i) {
    const int r = r_begin + i;
    if (r >= r_end) break;
    load_row(r + 1, dn);
    const size_t at = plane + static_cast<size_t>(r) * Wf + c0;
    float t[4], o[4];
    load4(target + at, t);
    const float lw = data_f * lat_w[r];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float x = mid[k + 1];
      const float ax = sgn(x - up[k + 1]) + sgn(x - dn[k + 1]) + sgn(x - mid[k]) + sgn(x - mid[k + 2]);
      const float dg = sgn(x - up[k]) + sgn(x - up[k + 2]) + sgn(x - dn[k]) + sgn(x - dn[k + 2]);
      o[k] = lw * (x - t[k]) + tv_f * (ax + dg * 0.70710678118654752440f);
    }
    if (EVEN || left >= 4) {
      __builtin_nontemporal_store(float4_any{o[0], o[1], o[2], o[3]}, reinterpret_cast<float4_any *>(d_pred + at));
    } else {
#pragma unroll
      for (int k = 0; k < 3; ++k)
        if (k < left) d_pred[at + k] = o[k];
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) { up[k] = mid[k]; mid[k] = dn[k]; }
  }
}

// ------------------------------------------------------------------ back end
// d_P[b, n, (c, i, j)] = d_y[b, c, py ps + i, px ps + j]  (transpose of un-patchify), stored as activation type
template <typename T>
__global__ __launch_bounds__(256) void patchify_act_kernel(const float *__restrict__ dy, T *__restrict__ dP, int64_t total,
                                                           int N, int Wp, int C, int ps, int sH, int sW) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= total) return;
  const int ho = C * ps * ps;
  const int64_t bn = e / ho;
  const int rem = static_cast<int>(e % ho);
  const int c = rem / (ps * ps), i = (rem / ps) % ps, j = rem % ps;
  const int64_t b = bn / N;
  const int n = static_cast<int>(bn % N), py = n / Wp, px = n % Wp;
  Act<T>::store(dP + e, dy[((b * C + c) * sH + py * ps + i) * sW + px * ps + j]);
}

// The same for patch sides that are multiples of four: a thread moves four neighbours of a fine row.
// Threads run over (four pixels, four patches side by side, patch row) fastest, so a wave reads
// whole 128-byte lines of a fine row and writes 128 contiguous bytes of each of its four patches.
template <typename T>
__global__ __launch_bounds__(256) void patchify_act4_kernel(const float *__restrict__ dy, T *__restrict__ dP, int64_t total4,
                                                            int Hp, int Wp, int C, int ps, int sH, int sW) {
  int64_t e = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (e >= total4) return;
  const int q = ps / 4, wq = (Wp + 3) / 4;
  const int j4 = static_cast<int>(e % q); e /= q;
  const int pxl = static_cast<int>(e % 4); e /= 4;
  const int i = static_cast<int>(e % ps); e /= ps;
  const int c = static_cast<int>(e % C); e /= C;
  const int pxh = static_cast<int>(e % wq); e /= wq;
  const int py = static_cast<int>(e % Hp);
  const int64_t b = e / Hp;
  const int px = pxh * 4 + pxl;
  if (px >= Wp) return;
  const float4 v = *reinterpret_cast<const float4 *>(dy + ((b * C + c) * sH + py * ps + i) * sW + px * ps + 4 * j4);
  T *o = dP + ((b * Hp + py) * static_cast<int64_t>(Wp) + px) * (static_cast<int64_t>(C) * ps * ps) + (c * ps + i) * ps + 4 * j4;
  if constexpr (std::is_same<T, float>::value) {
    *reinterpret_cast<float4 *>(o) = v;
  } else {
    const uint32_t lo = static_cast<uint32_t>(f32_to_bf16(v.x)) | (static_cast<uint32_t>(f32_to_bf16(v.y)) << 16);
    const uint32_t hi = static_cast<uint32_t>(f32_to_bf16(v.z)) | (static_cast<uint32_t>(f32_to_bf16(v.w)) << 16);
    *reinterpret_cast<uint2 *>(o) = make_uint2(lo, hi);
  }
}

// rows of the tile-major stream: an interior token takes its row of src[b, patch], a halo copy zero
__global__ __launch_bounds__(256) void scatter_interior_kernel(const float *__restrict__ src, const int32_t *__restrict__ gather,
                                                               const int32_t *__restrict__ interior_src, float *__restrict__ dst,
                                                               int64_t rows, int64_t n_h, int N, int D) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int64_t b = row / n_h;
  const int r = static_cast<int>(row % n_h);
  const int g = gather[r];
  const bool own = interior_src[g] == r;
  const float4 *in = reinterpret_cast<const float4 *>(src + (b * N + g) * D);
  float4 *out = reinterpret_cast<float4 *>(dst + row * D);
  for (int d = lane; d < D / 4; d += 64) out[d] = own ? in[d] : make_float4(0.f, 0.f, 0.f, 0.f);
}

// Gradient of the residual path's 3x3 convolution (weights and bias).  The forward evaluates
// R = b + sum over taps (dy, dx) and inputs i of w[o][i][dy][dx] U_i(r + dy, c + dx), U_i the bilinear
// upsampling of input i on the tile's haloed box (neighbours clamped to the box, zero outside it).
// U is linear in the coarse pixels, so with G_o the upstream gradient on a block of fine pixels
//   dw[o][i][dy][dx] = sum_{r,c} G_o(r, c) U_i(r + dy, c + dx) = sum_{Y,X} x_i(Y, X) Q[o][dy][dx](Y, X),
//   Q[o][dy][dx](Y, X) = sum_{r,c} G_o(r, c) RW[dy](Y, r) CW[dx](X, c),
// where RW[dy](Y, r) is the weight with which coarse row Y enters fine row r + dy (two non-zeros per
// fine row, zero for rows outside the box) and CW the same for columns: the upsampling transposed,
// rows first (P = RW G), then columns (Q = P CW^T), then one small product with the coarse window.
// That is 9 (C + about 2) multiply-adds per coarse-window pixel and output plus about 12 per fine pixel
// and output, instead of 9 C per fine pixel and output for the product with U written out, in fp32
// throughout.
//
// A work-group walks over 16 x 64 blocks of fine pixels (every block of every tile interior of every
// sample, dealt out in turn), CO = 4 OPT outputs per pass.  Row step: a thread owns one fine column
// and OPT outputs; for each coarse row it runs over the fine rows that touch it.  Column step: one
// thread per value of Q, over the fine columns that touch its coarse column.  Last step: one thread
// per (output, input) pair, nine sums over the window, added to the pair's accumulators in LDS (one
// owner per accumulator: a fixed order, no atomics).  One partial row of 9 C C + C sums per
// work-group; a fixed-order reduction follows.
struct ResGradArgs {
  const float *x, *dy;
  float *partial;
  const tile_desc *tiles;
  const int32_t *out_var_idx;
  int V, C, H, W, s, p, ps;
  int nbx, nby, T, batch;
  int cwh, cww;
};

constexpr size_t kResGradLds = 150 * 1024;        // dynamic LDS the kernel may ask for
// floats of dynamic LDS for CO outputs per pass
static size_t residual_wgrad_lds_floats(int C, int CO, int cwh, int cww) {
  const size_t npx = static_cast<size_t>(cwh) * cww;
  const size_t gq = std::max<size_t>(static_cast<size_t>(CO) * 16 * 64, (static_cast<size_t>(CO) * 9 * npx + 3) / 4 * 4);
  return gq + static_cast<size_t>(CO) * 3 * cwh * 64 + 3 * cwh * 16 + 3 * cww * 64 + C * npx + 9 * C * C + C + 6 * cww + 4;
}

// OPT: outputs per thread in the row step (CO = 4 OPT per pass).  NIT: the column step covers 4 NIT
// fine columns from the first one that touches a coarse column (a coarse column is touched by fewer
// than 2 s + 1 fine columns); a block where some run is longer takes all 64 columns instead.
template <int OPT, int NIT>
__global__ __launch_bounds__(256) void residual_wgrad_kernel(ResGradArgs a) {
  constexpr int BY = 16, BX = 64, WY = BY + 2, WX = BX + 2, WXP = 68, CO = 4 * OPT;
  __shared__ float row_w[WY], col_w[WXP];
  __shared__ int row_a[WY], row_b[WY], row_m[WY], col_a[WXP], col_b[WXP], col_m[WXP];
  __shared__ int var_idx[64];
  __shared__ int long_run;
  extern __shared__ __align__(16) float dynr[];
  const int cwh = a.cwh, cww = a.cww, npx = cwh * cww, qw = 3 * cww;
  const int gq = max(CO * BY * BX, (CO * 9 * npx + 3) / 4 * 4);   // a multiple of four: P and CW are read 16 bytes at a time
  float *G = dynr;                                // [CO][BY][BX] upstream gradient of the block ...
  float *Q = dynr;                                // ... later [CO][3][cwh][3][cww] (G is no longer needed by then)
  float *P = dynr + gq;                           // [CO][3][cwh][BX]
  float *RW = P + CO * 3 * cwh * BX;              // [3][cwh][BY]
  float *CW = RW + 3 * cwh * BY;                  // [3][cww][BX]
  float *Cw = CW + 3 * cww * BX;                  // [C][npx] coarse window of the inputs
  float *acc = Cw + a.C * npx;                    // [9 C C + C] accumulators of this work-group
  int *xlo = reinterpret_cast<int *>(acc + 9 * a.C * a.C + a.C), *xhi = xlo + qw;     // [3][cww] fine columns that touch coarse column X under tap dx
  const int t = threadIdx.x, lane = t & 63, og = t >> 6;
  const int n_acc = 9 * a.C * a.C + a.C;
  for (int i = t; i < n_acc; i += 256) acc[i] = 0.f;
  if (t < a.C) var_idx[t] = a.out_var_idx[t];
  const float inv_s = 1.0f / static_cast<float>(a.s);
  const int sH = a.s * a.H, sW = a.s * a.W;
  const int64_t blocks = static_cast<int64_t>(a.nbx) * a.nby * a.T * a.batch;
  auto src = [&](int f, int n_coarse, int &ia, int &ib, float &w1) {
    const float sc = (static_cast<float>(f) + 0.5f) * inv_s - 0.5f;
    const float fl = floorf(sc);
    w1 = sc - fl;
    const int i0 = static_cast<int>(fl);
    ia = min(max(i0, 0), n_coarse - 1);
    ib = min(max(i0 + 1, 0), n_coarse - 1);
  };
  for (int64_t blk = blockIdx.x; blk < blocks; blk += gridDim.x) {     // uniform over the work-group
    const int bxy = static_cast<int>(blk % (a.nbx * a.nby));
    const int tile = static_cast<int>((blk / (a.nbx * a.nby)) % a.T);
    const int b = static_cast<int>(blk / (static_cast<int64_t>(a.nbx) * a.nby * a.T));
    const tile_desc td = a.tiles[tile];
    const int ih = (td.y1 - td.y0) * a.ps, iw = (td.x1 - td.x0) * a.ps;
    const int iy0 = (bxy / a.nbx) * BY, ix0 = (bxy % a.nbx) * BX;
    if (iy0 >= ih || ix0 >= iw) continue;
    const int fy0 = (td.y0 - td.Y0) * a.ps + iy0, fx0 = (td.x0 - td.X0) * a.ps + ix0;
    const int box_fh = (td.Y1 - td.Y0) * a.ps, box_fw = (td.X1 - td.X0) * a.ps;
    const int box_ch = (td.Y1 - td.Y0) * a.p, box_cw = (td.X1 - td.X0) * a.p;
    const int cy_org = td.Y0 * a.p, cx_org = td.X0 * a.p;
    int oy, ox;
    {
      int ib_;
      float w_;
      src(fy0 - 1, box_ch, oy, ib_, w_);
      src(fx0 - 1, box_cw, ox, ib_, w_);
    }
    __syncthreads();                              // the previous block's tables and arrays are no longer read
    if (t < WY) {
      const int fy = fy0 + t - 1;
      int ia, ib;
      float w1;
      src(fy, box_ch, ia, ib, w1);
      row_a[t] = min(ia - oy, cwh - 1);
      row_b[t] = min(ib - oy, cwh - 1);
      row_w[t] = w1;
      row_m[t] = (fy >= 0 && fy < box_fh) ? 1 : 0;
    } else if (t >= 64 && t < 64 + WX) {
      const int wx = t - 64, fx = fx0 + wx - 1;
      int ia, ib;
      float w1;
      src(fx, box_cw, ia, ib, w1);
      col_a[wx] = min(ia - ox, cww - 1);
      col_b[wx] = min(ib - ox, cww - 1);
      col_w[wx] = w1;
      col_m[wx] = (fx >= 0 && fx < box_fw) ? 1 : 0;
    }
    if (t == 255) long_run = 0;
    if (t < qw) { xlo[t] = BX; xhi[t] = -1; }     // qw <= 3 * 68 < 256
    // coarse window of every input
    for (int idx = t; idx < a.C * npx; idx += 256) {
      const int ci = idx / npx, r = idx % npx;
      const int wy = r / cww, wx = r % cww;
      const float *xp = a.x + (static_cast<size_t>(b) * a.V + var_idx[ci]) * a.H * a.W;
      const int y = min(oy + wy, box_ch - 1), x = min(ox + wx, box_cw - 1);
      Cw[idx] = xp[static_cast<size_t>(cy_org + y) * a.W + cx_org + x];
    }
    __syncthreads();
    // transposed interpolation weights: RW[dy][Y][r] and CW[dx][X][c], window row r + dy / column c + dx
    for (int idx = t; idx < 3 * cwh * BY; idx += 256) {
      const int r = idx % BY, Y = (idx / BY) % cwh, dy = idx / (BY * cwh), wr = r + dy;
      const float w1 = row_w[wr];
      RW[idx] = row_m[wr] ? (row_a[wr] == Y ? 1.0f - w1 : 0.f) + (row_b[wr] == Y ? w1 : 0.f) : 0.f;
    }
    for (int idx = t; idx < 3 * cww * BX; idx += 256) {
      const int cc = idx % BX, e = idx / BX, X = e % cww, dx = e / cww, wc = cc + dx;
      const float w1 = col_w[wc];
      const float v = col_m[wc] ? (col_a[wc] == X ? 1.0f - w1 : 0.f) + (col_b[wc] == X ? w1 : 0.f) : 0.f;
      CW[idx] = v;
      if (v != 0.f) {
        atomicMin(&xlo[e], cc);
        atomicMax(&xhi[e], cc);
      }
    }
    __syncthreads();
    if (t < qw) {
      const int lo = min(xlo[t] & ~3, BX - 4 * NIT);            // 16-byte aligned start of the window of 4 NIT columns
      if (xhi[t] >= lo + 4 * NIT) long_run = 1;
      xlo[t] = lo;
    }
    for (int co0 = 0; co0 < a.C; co0 += CO) {
      const int nco = min(CO, a.C - co0);
      __syncthreads();                            // Q of the previous pass consumed (and the run tables written)
      // upstream gradient of the block, zero past the interior's edge and for outputs past the last
      for (int e = t; e < CO * BY * BX / 4; e += 256) {
        const int o = e / (BY * BX / 4), yy = (e / (BX / 4)) % BY, xx = 4 * (e % (BX / 4));
        const int iy = iy0 + yy, ix = ix0 + xx;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (o < nco && iy < ih) {
          const float *gp = a.dy + ((static_cast<size_t>(b) * a.C + co0 + o) * sH + td.y0 * a.ps + iy) * sW + td.x0 * a.ps + ix;
          if (ix + 3 < iw && (reinterpret_cast<uintptr_t>(gp) & 15) == 0) {
            v = *reinterpret_cast<const float4 *>(gp);
          } else {
            if (ix < iw) v.x = gp[0];
            if (ix + 1 < iw) v.y = gp[1];
            if (ix + 2 < iw) v.z = gp[2];
            if (ix + 3 < iw) v.w = gp[3];
          }
        }
        *reinterpret_cast<float4 *>(G + (o * BY + yy) * BX + xx) = v;
      }
      __syncthreads();
      // rows: P[o][dy][Y][c] = sum_r RW[dy][Y][r] G[o][r][c]; the bias gradient is the plain sum of G.
      // A thread keeps its column of G for its OPT outputs in registers over all coarse rows.
      {
        float gcol[OPT][BY], bs[OPT];
#pragma unroll
        for (int j = 0; j < OPT; ++j) {
          bs[j] = 0.f;
#pragma unroll
          for (int r = 0; r < BY; ++r) {
            gcol[j][r] = G[((og * OPT + j) * BY + r) * BX + lane];
            bs[j] += gcol[j][r];
          }
        }
        for (int Y = 0; Y < cwh; ++Y) {
          float s3[OPT][3];
#pragma unroll
          for (int j = 0; j < OPT; ++j) s3[j][0] = s3[j][1] = s3[j][2] = 0.f;
#pragma unroll
          for (int r = 0; r < BY; ++r) {
            const float c0 = RW[Y * BY + r], c1 = RW[(cwh + Y) * BY + r], c2 = RW[(2 * cwh + Y) * BY + r];
#pragma unroll
            for (int j = 0; j < OPT; ++j) {
              s3[j][0] = fmaf(gcol[j][r], c0, s3[j][0]);
              s3[j][1] = fmaf(gcol[j][r], c1, s3[j][1]);
              s3[j][2] = fmaf(gcol[j][r], c2, s3[j][2]);
            }
          }
#pragma unroll
          for (int j = 0; j < OPT; ++j)
#pragma unroll
            for (int d = 0; d < 3; ++d) P[(((og * OPT + j) * 3 + d) * cwh + Y) * BX + lane] = s3[j][d];
        }
        // a wave holds one group of OPT outputs: add its 64 columns, lane 0 owns the accumulators
#pragma unroll
        for (int j = 0; j < OPT; ++j) {
          float v = bs[j];
          for (int w = 1; w < 64; w <<= 1) v += __shfl_xor(v, w);
          if (lane == 0 && og * OPT + j < nco) acc[9 * a.C * a.C + co0 + og * OPT + j] += v;
        }
      }
      __syncthreads();                            // P written, G no longer read: Q may overwrite it
      // columns: Q[row = (o, dy, Y)][dx][X] = sum_c CW[dx][X][c] P[row][c] over the window of columns that
      // holds the run of (dx, X) (the weights outside a run are zero)
      {
        const int nrows = CO * 3 * cwh, rstep = 256 / qw;
        const int e = t % qw, r0 = t / qw;        // a thread keeps its (dx, X); threads past the last multiple of qw rest
        const bool whole = long_run != 0;         // uniform
        const float4 *cp = reinterpret_cast<const float4 *>(CW + e * BX);
        if (r0 < rstep && !whole) {
          const int lo4 = xlo[e] >> 2;
          float4 cw4[NIT];
#pragma unroll
          for (int i = 0; i < NIT; ++i) cw4[i] = cp[lo4 + i];
          for (int row = r0; row < nrows; row += rstep) {
            const float4 *pp = reinterpret_cast<const float4 *>(P + row * BX) + lo4;
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < NIT; ++i) {
              const float4 pv = pp[i];
              sum = fmaf(pv.x, cw4[i].x, sum);
              sum = fmaf(pv.y, cw4[i].y, sum);
              sum = fmaf(pv.z, cw4[i].z, sum);
              sum = fmaf(pv.w, cw4[i].w, sum);
            }
            Q[row * qw + e] = sum;
          }
        } else if (r0 < rstep) {
          for (int row = r0; row < nrows; row += rstep) {
            const float4 *pp = reinterpret_cast<const float4 *>(P + row * BX);
            float sum = 0.f;
#pragma unroll
            for (int i = 0; i < BX / 4; ++i) {
              const float4 pv = pp[i], cv = cp[i];
              sum = fmaf(pv.x, cv.x, sum);
              sum = fmaf(pv.y, cv.y, sum);
              sum = fmaf(pv.z, cv.z, sum);
              sum = fmaf(pv.w, cv.w, sum);
            }
            Q[row * qw + e] = sum;
          }
        }
      }
      __syncthreads();
      // window: dw[o][i][dy][dx] += sum_{Y,X} x_i(Y, X) Q[(o, dy, Y)][dx][X]
      for (int pr = t; pr < nco * a.C; pr += 256) {
        const int o = pr / a.C, ci = pr % a.C;
        const float *xw = Cw + ci * npx;
        float s9[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) s9[k] = 0.f;
        for (int Y = 0; Y < cwh; ++Y) {
          const float *q0 = Q + ((o * 3 + 0) * cwh + Y) * qw, *q1 = Q + ((o * 3 + 1) * cwh + Y) * qw, *q2 = Q + ((o * 3 + 2) * cwh + Y) * qw;
#pragma unroll 4
          for (int X = 0; X < cww; ++X) {
            const float xv = xw[Y * cww + X];
            s9[0] = fmaf(xv, q0[X], s9[0]); s9[1] = fmaf(xv, q0[cww + X], s9[1]); s9[2] = fmaf(xv, q0[2 * cww + X], s9[2]);
            s9[3] = fmaf(xv, q1[X], s9[3]); s9[4] = fmaf(xv, q1[cww + X], s9[4]); s9[5] = fmaf(xv, q1[2 * cww + X], s9[5]);
            s9[6] = fmaf(xv, q2[X], s9[6]); s9[7] = fmaf(xv, q2[cww + X], s9[7]); s9[8] = fmaf(xv, q2[2 * cww + X], s9[8]);
          }
        }
        float *ap = acc + ((co0 + o) * a.C + ci) * 9;
#pragma unroll
        for (int k = 0; k < 9; ++k) ap[k] += s9[k];
      }
    }
  }
  __syncthreads();
  for (int i = t; i < n_acc; i += 256) a.partial[static_cast<size_t>(blockIdx.x) * n_acc + i] = acc[i];
}

// ------------------------------------------------------------------ front end
// d_z[b, g, :] = sum over the tile-major copies of patch g (listed in increasing index: a fixed order)
template <typename T>
__global__ __launch_bounds__(256) void gather_transpose_kernel(const float *__restrict__ d_tok, const int32_t *__restrict__ off,
                                                               const int32_t *__restrict__ idx, float *__restrict__ d_z,
                                                               T *__restrict__ d_z_act, int64_t rows, int64_t n_h, int N, int D) {
  const int lane = threadIdx.x & 63;
  const int64_t row = static_cast<int64_t>(blockIdx.x) * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int64_t b = row / N;
  const int g = static_cast<int>(row % N);
  const int lo = off[g], hi = off[g + 1];
  for (int d = lane * 4; d < D; d += 256) {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = lo; k < hi; ++k) {
      const float4 v = *reinterpret_cast<const float4 *>(d_tok + (b * n_h + idx[k]) * D + d);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    *reinterpret_cast<float4 *>(d_z + row * D + d) = s;
    T *o = d_z_act + row * D + d;
    Act<T>::store(o, s.x); Act<T>::store(o + 1, s.y); Act<T>::store(o + 2, s.z); Act<T>::store(o + 3, s.w);
  }
}

// out[n] = sum_b in[b * stride + n] (samples added in increasing order)
__global__ __launch_bounds__(256) void batch_sum_kernel(const float *__restrict__ in, float *__restrict__ out, int64_t n,
                                                        int64_t stride, int batch) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= n) return;
  float s = 0.f;
  for (int b = 0; b < batch; ++b) s += in[b * stride + i];
  out[i] = s;
}

// Folded tokenisation + aggregation, backwards, first half: per token and head the softmax over
// the variables a[g, v] (recomputed as in the forward) and the gradient of its logits
//   d_s[g, v] = a[g, v] (d_a[g, v] - sum_v' a[g, v'] d_a[g, v']),  d_a[g, v] = sum_{d in head g} d_o[d] val[v, d],
//   val[v, d] = U[v, d, :] . pixels_v + c[v, d].
// The sums over the head's features do not depend on the pixels:
//   d_a[g, v] = sum_i pixels_v[i] E[(g, v, i)] + E[(g, v, p2)],  E[(g, v, j)] = sum_{d in head g} d_o[d] (U[v, d, j] | c[v, d]),
// so E = d_o W^T is one GEMM over all tokens with the block-structured table W[(g, v, j), d] (zero
// where d is outside head g: the matrix unit does heads times the needed products and is still far
// quicker than the vector units on the plain form), and this kernel only combines E with the pixels.
struct AggBwdArgs {
  const float *x, *A, *a0;
  const void *d_o;            // act [BN, D]
  const float *E;             // [BN, ne] rows (g, v, j), j <= p2
  float *a_out;               // [BN, heads, V] softmax weights
  float *x_out;               // [BN, V (p2 + 1)] pixels of a token by variable, each variable's followed by a one
  float *partial;             // [gridDim.x, V, p2 + 1, heads] sums over a work-group's tokens of d_s times those
  int V, H, W, p, Wp, N, D, heads, dh, ne;
  int64_t BN;
};

// W[(g * V + v) * (p2 + 1) + j][d] = U[v][d][j] (j < p2) or c[v][d] (j = p2) for d in head g, else 0; rows past the last: 0
template <typename T>
__global__ __launch_bounds__(256) void agg_value_table_kernel(const float *__restrict__ U, const float *__restrict__ cc, T *__restrict__ Wt,
                                                              int V, int D, int dh, int p2, int rows, int ne) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= static_cast<int64_t>(ne) * D) return;
  const int d = static_cast<int>(i % D), r = static_cast<int>(i / D);
  float val = 0.f;
  if (r < rows) {
    const int j = r % (p2 + 1), gv = r / (p2 + 1), v = gv % V, g = gv / V;
    if (d / dh == g) val = j < p2 ? U[(static_cast<size_t>(v) * D + d) * p2 + j] : cc[static_cast<size_t>(v) * D + d];
  }
  Act<T>::store(Wt + i, val);
}

// A work-group takes groups of TP tokens in turn.  The gradients of the folded score tables, dA[v, g, i] = sum over the
// tokens of d_s[g, v] pixels_v[i] and da0[v, g] = sum of d_s[g, v], are formed right here, where both factors lie in LDS:
// thread = (variable, head), added to the work-group's own partial row (written by its first group).
template <int TP, int p2>
__global__ __launch_bounds__(256) void agg_scores_bwd_kernel(AggBwdArgs e) {
  extern __shared__ __align__(16) float smg[];
  constexpr int P3 = p2 + 1;
  const int VP2 = e.V * p2, HV = e.heads * e.V, VP3 = e.V * P3;
  float *pix = smg;                        // [TP][V*p2]
  float *sc = pix + TP * VP2;              // [TP][heads][V] logits, then softmax weights
  float *da = sc + TP * HV;                // [TP][heads][V] gradients of the weights, then of the logits
  const int t = threadIdx.x;
  float *part = e.partial + static_cast<size_t>(blockIdx.x) * VP3 * e.heads;
  const int64_t groups = (e.BN + TP - 1) / TP;
  for (int64_t grp = blockIdx.x; grp < groups; grp += gridDim.x) {
    const int64_t bn0 = grp * TP;
    __syncthreads();                       // the previous group's values are no longer read
    for (int idx = t; idx < TP * VP2; idx += 256) {
      const int pi = idx / VP2, rem = idx % VP2, v = rem / p2, i = rem % p2;
      const int64_t bn = bn0 + pi;
      float val = 0.f;
      if (bn < e.BN) {
        const int64_t b = bn / e.N;
        const int n = static_cast<int>(bn % e.N);
        const int py = n / e.Wp, px = n % e.Wp;
        val = e.x[((b * e.V + v) * e.H + py * e.p + i / e.p) * e.W + px * e.p + i % e.p];
      }
      pix[idx] = val;
    }
    __syncthreads();
    for (int idx = t; idx < TP * VP3; idx += 256) {
      const int pi = idx / VP3, rem = idx % VP3, v = rem / P3, i = rem % P3;
      if (bn0 + pi < e.BN) e.x_out[bn0 * VP3 + idx] = i < p2 ? pix[pi * VP2 + v * p2 + i] : 1.0f;
    }
    // logits, and d_a from E: consecutive threads read consecutive (p2 + 1)-float groups of a row of E
    for (int idx = t; idx < TP * HV; idx += 256) {
      const int pi = idx / HV, gv = idx % HV, g = gv / e.V, v = gv % e.V;
      const int64_t bn = bn0 + pi;
      const float *Ar = e.A + (static_cast<size_t>(v) * e.heads + g) * p2;
      const float *px = pix + pi * VP2 + v * p2;
      float s = e.a0[v * e.heads + g], dv = 0.f;
#pragma unroll
      for (int i = 0; i < p2; ++i) s = fmaf(Ar[i], px[i], s);
      if (bn < e.BN) {
        const float *er = e.E + bn * e.ne + static_cast<size_t>(gv) * P3;
        dv = er[p2];
#pragma unroll
        for (int i = 0; i < p2; ++i) dv = fmaf(px[i], er[i], dv);
      }
      sc[idx] = s;
      da[idx] = dv;
    }
    __syncthreads();
    for (int idx = t; idx < TP * e.heads; idx += 256) {
      float *r = sc + static_cast<size_t>(idx) * e.V, *dr = da + static_cast<size_t>(idx) * e.V;
      float mx = -INFINITY;
      for (int v = 0; v < e.V; ++v) mx = fmaxf(mx, r[v]);
      float sum = 0.f, dot = 0.f;
      for (int v = 0; v < e.V; ++v) {
        const float ex = __expf(r[v] - mx);
        r[v] = ex;
        sum += ex;
        dot = fmaf(ex, dr[v], dot);
      }
      const float inv = 1.0f / sum;
      dot *= inv;
      for (int v = 0; v < e.V; ++v) {
        const float w = r[v] * inv;
        r[v] = w;
        dr[v] = w * (dr[v] - dot);
      }
    }
    __syncthreads();
    for (int idx = t; idx < TP * HV; idx += 256)
      if (bn0 + idx / HV < e.BN) e.a_out[bn0 * HV + idx] = sc[idx];
    const int have = static_cast<int>(min(static_cast<int64_t>(TP), e.BN - bn0));
    const bool first = grp == blockIdx.x;
    for (int item = t; item < HV; item += 256) {
      const int v = item / e.heads, g = item % e.heads;
      float acc[P3];
      float *o = part + static_cast<size_t>(v) * P3 * e.heads + g;
#pragma unroll
      for (int i = 0; i <= p2; ++i) acc[i] = first ? 0.f : o[static_cast<size_t>(i) * e.heads];
      for (int pi = 0; pi < have; ++pi) {
        const float ds = da[(pi * e.heads + g) * e.V + v];
        const float *px = pix + pi * VP2 + v * p2;
#pragma unroll
        for (int i = 0; i < p2; ++i) acc[i] = fmaf(ds, px[i], acc[i]);
        acc[p2] += ds;
      }
#pragma unroll
      for (int i = 0; i <= p2; ++i) o[static_cast<size_t>(i) * e.heads] = acc[i];
    }
  }
}

// Second half: gradients of the folded value tables, for head g
//   T[(v, i), d] = sum over tokens of (a[g, v] xt[v, i]) d_o[d],  xt = the pixels of variable v, then one,
// a product over the tokens per head, on fp32 matrix instructions (32x32x2: two tokens each, the first factor
// multiplied together in the lane that holds its row).  Grid (token slab, head and 64 of its features, 32 MB rows);
// the four waves take every fourth pair of tokens and meet in LDS in wave order.  One partial table [V (p2 + 1), D]
// per slab.  c2 with one sample (64,800 tokens): 1.24 ms with one thread per feature reading every factor, 0.25 here.
template <typename T, int MB>
__global__ __launch_bounds__(256) void agg_values_bwd_kernel(AggBwdArgs e, float *__restrict__ partial, int tokens_per_slab, int chunks) {
  typedef __attribute__((ext_vector_type(16))) float f32x16;
  constexpr int NB = 2, AHEAD = 4;
  __shared__ float box[3][16][64];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hi = lane >> 5;
  const int P3 = e.p * e.p + 1, rows = e.V * P3, HV = e.heads * e.V;
  const int g = blockIdx.y / chunks, f0 = (blockIdx.y % chunks) * 64, m0 = blockIdx.z * MB * 32;
  const int64_t t0 = static_cast<int64_t>(blockIdx.x) * tokens_per_slab, t1 = min(t0 + tokens_per_slab, e.BN);
  const T *dop = static_cast<const T *>(e.d_o) + g * e.dh;
  int m[MB], va[MB], f[NB];
#pragma unroll
  for (int k = 0; k < MB; ++k) {
    m[k] = min(m0 + k * 32 + l32, rows - 1);           // rows past the table repeat the last one and are not stored
    va[k] = g * e.V + m[k] / P3;
  }
#pragma unroll
  for (int n = 0; n < NB; ++n) f[n] = min(f0 + n * 32 + l32, e.dh - 1);
  f32x16 acc[MB][NB] = {};
  float xr[AHEAD][MB], ar[AHEAD][MB], br[AHEAD][NB];
  auto fetch = [&](int i, int64_t at) {                // tokens at, at + 1 of the two lane halves; zeros past the slab
    const int64_t tok = at + hi, c = min(tok, t1 - 1);
    const bool in = tok < t1;
#pragma unroll
    for (int k = 0; k < MB; ++k) {
      xr[i][k] = e.x_out[c * rows + m[k]];
      ar[i][k] = e.a_out[c * HV + va[k]];
    }
#pragma unroll
    for (int n = 0; n < NB; ++n) br[i][n] = in ? Act<T>::load(dop + c * e.D + f[n]) : 0.f;
  };
  const int64_t first = t0 + 2 * wave;
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) fetch(i, first + 8 * i);
  for (int64_t at = first; at < t1; at += 8 * AHEAD) {
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      float av[MB], bv[NB];
#pragma unroll
      for (int k = 0; k < MB; ++k) av[k] = xr[i][k] * ar[i][k];
#pragma unroll
      for (int n = 0; n < NB; ++n) bv[n] = br[i][n];
      fetch(i, at + 8 * (AHEAD + i));
#pragma unroll
      for (int k = 0; k < MB; ++k)
#pragma unroll
        for (int n = 0; n < NB; ++n) acc[k][n] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[k], bv[n], acc[k][n], 0, 0, 0);
    }
  }
  float *out = partial + static_cast<size_t>(blockIdx.x) * rows * e.D + g * e.dh;
#pragma unroll
  for (int k = 0; k < MB; ++k)
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      __syncthreads();
      if (wave > 0)
#pragma unroll
        for (int r = 0; r < 16; ++r) box[wave - 1][r][lane] = acc[k][n][r];
      __syncthreads();
      if (wave == 0 && f0 + n * 32 + l32 < e.dh)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + k * 32 + 8 * (r / 4) + 4 * hi + r % 4;
          if (row < rows) out[static_cast<size_t>(row) * e.D + f0 + n * 32 + l32] = ((acc[k][n][r] + box[0][r][lane]) + box[1][r][lane]) + box[2][r][lane];
        }
    }
}

// ---- Chain rule through the fold (fp32, small).  With the offsets as one more pixel, i = p2,
//   Wt[(v, i), j] = W_pe[v][j, i] | t_v[j] = b_pe[v] + var_emb[v],   tU[(v, i), d] = dU[v][d, i] | dc[v][d],
//   tA[(v, i), g] = dA[v, g, i] | da0[v, g],   q = Wq q0 + bq,   r[g, j] = kappa sum_{d in g} q[d] Wk[d, j],
// the forward is A = r Wt per head, U = Wv Wt (+ bv), so
//   d_r = tA^T Wt,   d_Wv = tU^T Wt,   d_Wt = tA r + tU Wv   (rows i < p2: d_W_pe, row p2: d_b_pe = d_var_emb).
// Three products for all variables at once; one variable after the other they were 6 V launches of a few microseconds
// (1.5 of the 5.6 ms of a step of the 9.5M model, about 6 of 125 ms at c2).
struct FoldArgs {
  const float *w_pe, *b_pe, *var_emb, *q0, *wq, *bq, *wk, *bk, *wv, *tU, *tA, *agg_bo_grad;
  float *q, *r, *Wt, *d_r, *d_q;
  float *g_w_pe, *g_b_pe, *g_var_emb, *g_wv, *g_bv, *g_wk, *g_bk, *g_wq, *g_bq, *g_q0, *g_res;
  int V, D, dh, heads, p2, n_res, res_idx;
  float kappa;
};

__device__ __forceinline__ float wave_total(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// q (one wave per row of Wq), Wt, the bias of the values and the resolution table's gradient (one row is the output
// map's bias gradient, the others are zero)
__global__ __launch_bounds__(256) void fold_prepare_kernel(FoldArgs a, int q_blocks) {
  const int P3 = a.p2 + 1;
  if (static_cast<int>(blockIdx.x) < q_blocks) {
    const int d = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (d >= a.D) return;
    const float *w = a.wq + static_cast<size_t>(d) * a.D;
    float s = 0.f;
    for (int j = lane; j < a.D; j += 64) s = fmaf(w[j], a.q0[j], s);
    s = wave_total(s);
    if (lane == 0) a.q[d] = s + a.bq[d];
    return;
  }
  const int64_t i = static_cast<int64_t>(blockIdx.x - q_blocks) * 256 + threadIdx.x;
  const int64_t n_wt = static_cast<int64_t>(a.V) * P3 * a.D;
  if (i < n_wt) {
    const int j = static_cast<int>(i % a.D), k = static_cast<int>(i / a.D), v = k / P3, pi = k % P3;
    const size_t vj = static_cast<size_t>(v) * a.D + j;
    a.Wt[i] = pi < a.p2 ? a.w_pe[vj * a.p2 + pi] : a.b_pe[vj] + a.var_emb[vj];
    return;
  }
  const int64_t k = i - n_wt;
  if (k < a.D) {
    float s = 0.f;
    for (int v = 0; v < a.V; ++v) s += a.tU[(static_cast<size_t>(v) * P3 + a.p2) * a.D + k];
    a.g_bv[k] = s;
  } else if (k < a.D + static_cast<int64_t>(a.n_res) * a.D) {
    const int64_t o = k - a.D;
    a.g_res[o] = o / a.D == a.res_idx ? a.agg_bo_grad[o % a.D] : 0.f;
  }
}

// r[g, j]: 64 columns per work-group, four row groups of the head added in order
__global__ __launch_bounds__(256) void fold_query_kernel(FoldArgs a) {
  __shared__ float box[4][64];
  const int g = blockIdx.y, col = threadIdx.x & 63, part = threadIdx.x >> 6, j = blockIdx.x * 64 + col;
  float s = 0.f;
  if (j < a.D)
    for (int d = part; d < a.dh; d += 4) s = fmaf(a.q[g * a.dh + d], a.wk[static_cast<size_t>(g * a.dh + d) * a.D + j], s);
  box[part][col] = s;
  __syncthreads();
  if (part == 0 && j < a.D) a.r[static_cast<size_t>(g) * a.D + j] = a.kappa * ((box[0][col] + box[1][col]) + (box[2][col] + box[3][col]));
}

// One 32 x 32 tile of a product per work-group, on fp32 matrix instructions; its four waves take every fourth step of
// two k and meet in LDS in wave order.  tile < n1: d_Wv; < n1 + n2: d_Wt; else d_r.
__global__ __launch_bounds__(256) void fold_products_kernel(FoldArgs a, int n1, int n2, int cols) {
  typedef __attribute__((ext_vector_type(16))) float f32x16;
  __shared__ float box[3][16][64];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6), l32 = lane & 31, hi = lane >> 5;
  const int rows3 = a.V * (a.p2 + 1), id = blockIdx.x;
  const int kind = id < n1 ? 0 : id < n1 + n2 ? 1 : 2, tile = kind == 0 ? id : kind == 1 ? id - n1 : id - n1 - n2;
  const int m0 = tile / cols * 32, n0 = tile % cols * 32, n = min(n0 + l32, a.D - 1);
  const int M = kind == 0 ? a.D : kind == 1 ? rows3 : a.heads;
  const int m = min(m0 + l32, M - 1);
  f32x16 acc = {};
  // A[m, k] at pa + k * ska, B[k, n] at pb + k * a.D
  auto run = [&](const float *pa, size_t ska, const float *pb, int K) {
    for (int s = wave; 2 * s < K; s += 32) {             // eight steps' factors at a time
      float x[8], y[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = 2 * (s + 4 * i) + hi, kc = min(k, K - 1);
        x[i] = pa[kc * ska];
        y[i] = pb[static_cast<size_t>(kc) * a.D];
        if (k >= K) x[i] = 0.f;
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i], y[i], acc, 0, 0, 0);
    }
  };
  if (kind == 0) {
    run(a.tU + m, a.D, a.Wt + n, rows3);
  } else if (kind == 1) {
    run(a.tA + static_cast<size_t>(m) * a.heads, 1, a.r + n, a.heads);
    run(a.tU + static_cast<size_t>(m) * a.D, 1, a.wv + n, a.D);
  } else {
    run(a.tA + m, a.heads, a.Wt + n, rows3);
  }
  if (wave > 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) box[wave - 1][r][lane] = acc[r];
  __syncthreads();
  if (wave > 0 || n0 + l32 >= a.D) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = m0 + 8 * (r / 4) + 4 * hi + r % 4, col = n0 + l32;
    if (row >= M) continue;
    const float v = ((acc[r] + box[0][r][lane]) + box[1][r][lane]) + box[2][r][lane];
    if (kind == 0) {
      a.g_wv[static_cast<size_t>(row) * a.D + col] = v;
    } else if (kind == 2) {
      a.d_r[static_cast<size_t>(row) * a.D + col] = v;
    } else {
      const int var = row / (a.p2 + 1), i = row % (a.p2 + 1);
      const size_t vj = static_cast<size_t>(var) * a.D + col;
      if (i < a.p2) {
        a.g_w_pe[vj * a.p2 + i] = v;
      } else {
        a.g_b_pe[vj] = v;
        a.g_var_emb[vj] = v;
      }
    }
  }
}

// the key and query ends of the fold: d_wk[d, j] = kappa q[d] d_r[head(d), j];  d_bk[d] = kappa q[d] s0[head(d)];
// d_q[d] = kappa (wk[d, :] . d_r[head(d), :] + bk[d] s0[head(d)]),  s0[g] = sum_v da0[v, g];  d_wq[d, j] = d_q[d] q0[j]
__global__ __launch_bounds__(256) void fold_key_bwd_kernel(FoldArgs a) {
  const int d = blockIdx.x, g = d / a.dh;         // one work-group per feature d
  __shared__ float red[4];
  const float kq = a.kappa * a.q[d];
  const float *dr = a.d_r + static_cast<size_t>(g) * a.D, *wk = a.wk + static_cast<size_t>(d) * a.D;
  float s = 0.f;
  for (int j = threadIdx.x; j < a.D; j += 256) {
    const float v = dr[j];
    a.g_wk[static_cast<size_t>(d) * a.D + j] = kq * v;
    s = fmaf(wk[j], v, s);
  }
  s = wave_total(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  float s0 = 0.f;
  for (int v = 0; v < a.V; ++v) s0 += a.tA[(static_cast<size_t>(v) * (a.p2 + 1) + a.p2) * a.heads + g];
  __syncthreads();
  const float dq = a.kappa * (((red[0] + red[1]) + (red[2] + red[3])) + a.bk[d] * s0);
  if (threadIdx.x == 0) {
    a.g_bk[d] = kq * s0;
    a.d_q[d] = dq;
    a.g_bq[d] = dq;
  }
  for (int j = threadIdx.x; j < a.D; j += 256) a.g_wq[static_cast<size_t>(d) * a.D + j] = dq * a.q0[j];
}

// d_q0[j] = sum_d Wq[d, j] d_q[d]: 64 columns per work-group, sixteen row groups added in order
__global__ __launch_bounds__(1024) void fold_q0_kernel(FoldArgs a) {
  __shared__ float box[16][64];
  const int col = threadIdx.x & 63, part = threadIdx.x >> 6, j = blockIdx.x * 64 + col;
  float s = 0.f;
  if (j < a.D)
    for (int d = part; d < a.D; d += 16) s = fmaf(a.wq[static_cast<size_t>(d) * a.D + j], a.d_q[d], s);
  box[part][col] = s;
  __syncthreads();
  if (part == 0 && j < a.D) {
    float v = box[0][col];
#pragma unroll
    for (int k = 1; k < 16; ++k) v += box[k][col];
    a.g_q0[j] = v;
  }
}

// ------------------------------------------------------------------ buffers
struct HeadWs {
  void *dP, *Af, *dAf;       // act [Mi, head_out], [Mi, D], [Mi, D]
  float *Xi, *dXi;           // [Mi, D]
  void *wgrad;
  float *lnp, *resp;         // partial rows: LayerNorm parameters, residual path
  int res_wg;
  size_t total;
};
static int residual_grid(const reslim_ctx *c, int batch, int *nbx, int *nby) {
  int max_ih = 0, max_iw = 0;
  for (const tile_desc &t : c->tiles) {
    max_ih = std::max(max_ih, (t.y1 - t.y0) * c->ps);
    max_iw = std::max(max_iw, (t.x1 - t.x0) * c->ps);
  }
  *nbx = (max_iw + 63) / 64;
  *nby = (max_ih + 15) / 16;
  const int64_t blocks = static_cast<int64_t>(*nbx) * *nby * c->T * batch;
  return static_cast<int>(std::min<int64_t>(blocks, 768));
}
static HeadWs plan_head_ws(const reslim_ctx *c, int batch, void *base) {
  const size_t Mi = static_cast<size_t>(batch) * c->N, D = c->cfg.embed_dim, es = act_size(c), ho = c->head_out;
  unsigned char *p = static_cast<unsigned char *>(base);
  size_t off = 0;
  auto take = [&](size_t bytes) { unsigned char *q = p + off; off += align256(bytes); return q; };
  HeadWs w;
  w.dP = take(Mi * ho * es);
  w.Af = take(Mi * D * es);
  w.dAf = take(Mi * D * es);
  w.Xi = reinterpret_cast<float *>(take(Mi * D * 4));
  w.dXi = reinterpret_cast<float *>(take(Mi * D * 4));
  const WgradOp op = {nullptr, nullptr, nullptr, nullptr, c->head_out, c->cfg.embed_dim};
  w.wgrad = take(std::max<size_t>(wgrad_ws_bytes(c->cfg.dtype, &op, 1, static_cast<int>(Mi)), 256));
  w.lnp = reinterpret_cast<float *>(take(static_cast<size_t>(layernorm_bwd_slabs(Mi)) * 2 * D * 4));
  int nbx, nby;
  w.res_wg = residual_grid(c, batch, &nbx, &nby);
  const size_t C = c->cfg.out_vars;
  w.resp = reinterpret_cast<float *>(take(static_cast<size_t>(w.res_wg) * (9 * C * C + C) * 4));
  w.total = off;
  return w;
}

// rows of the value table of the aggregation gradient's GEMM: (head, variable, pixel | offset), a multiple of 8
static int agg_table_rows(const reslim_ctx *c) {
  return (c->cfg.heads * c->cfg.in_vars * (c->cfg.patch * c->cfg.patch + 1) + 7) / 8 * 8;
}
struct EmbedWs {
  float *dz;                 // [Mi, D]
  void *dz_act, *o, *d_o;    // act [Mi, D]: gradient of the aggregated tokens, aggregated values, their gradient
  void *wgrad;
  float *a, *xt;             // [Mi, heads, V] softmax weights, [Mi, V (p2 + 1)] pixels
  float *E;                  // [Mi, n_e] d_o times the block-structured value table
  float *pU, *pA;            // partial rows of the folded tables' gradients
  float *tU, *tA;            // reduced tables [V, p2 + 1, D], [V, p2 + 1, heads]
  float *q, *r, *Wt, *d_r, *d_q;   // fold intermediates: [D], [heads, D], [V, p2 + 1, D], [heads, D], [D]
  int slabs_u, tok_u, mb_u, slabs_a, tp;
  size_t lds_a, total;
};
static EmbedWs plan_embed_ws(const reslim_ctx *c, int batch, void *base) {
  const size_t Mi = static_cast<size_t>(batch) * c->N, D = c->cfg.embed_dim, es = act_size(c);
  const size_t V = c->cfg.in_vars, heads = c->cfg.heads, p2 = static_cast<size_t>(c->cfg.patch) * c->cfg.patch;
  unsigned char *p = static_cast<unsigned char *>(base);
  size_t off = 0;
  auto take = [&](size_t bytes) { unsigned char *q = p + off; off += align256(bytes); return q; };
  EmbedWs w;
  w.dz = reinterpret_cast<float *>(take(Mi * D * 4));
  w.dz_act = take(Mi * D * es);
  w.o = take(Mi * D * es);
  w.d_o = take(Mi * D * es);
  const WgradOp op = {nullptr, nullptr, nullptr, nullptr, c->cfg.embed_dim, c->cfg.embed_dim};
  w.wgrad = take(std::max<size_t>(wgrad_ws_bytes(c->cfg.dtype, &op, 1, static_cast<int>(Mi)), 256));
  w.a = reinterpret_cast<float *>(take(Mi * heads * V * 4));
  w.xt = reinterpret_cast<float *>(take(Mi * V * (p2 + 1) * 4));
  w.E = reinterpret_cast<float *>(take(Mi * static_cast<size_t>(agg_table_rows(c)) * 4));
  // value tables: row blocks of 32 per work-group (up to four), then as many token slabs as give about four work-groups
  // per CU, at least 64 tokens each
  const size_t blocks = (V * (p2 + 1) + 31) / 32, z = (blocks + 3) / 4;
  w.mb_u = static_cast<int>((blocks + z - 1) / z);
  const size_t per = heads * ((static_cast<size_t>(c->dh) + 63) / 64) * z;
  const size_t su = std::min(std::max<size_t>(1, std::min<size_t>(256, 1024 / per)), (Mi + 63) / 64);
  w.tok_u = static_cast<int>((Mi + su - 1) / su);
  w.slabs_u = static_cast<int>((Mi + w.tok_u - 1) / w.tok_u);
  // score tables: tokens per group by what fits LDS, at most 512 work-groups (their partial rows are added afterwards)
  auto lds_for = [&](size_t tp) { return tp * (V * p2 + 2 * heads * V) * sizeof(float); };
  w.tp = lds_for(16) <= 64 * 1024 ? 16 : 4;
  w.lds_a = lds_for(w.tp);
  w.slabs_a = static_cast<int>(std::min<size_t>(512, (Mi + w.tp - 1) / w.tp));
  w.pU = reinterpret_cast<float *>(take(static_cast<size_t>(w.slabs_u) * V * D * (p2 + 1) * 4));
  w.pA = reinterpret_cast<float *>(take(static_cast<size_t>(w.slabs_a) * V * heads * (p2 + 1) * 4));
  w.tU = reinterpret_cast<float *>(take(V * D * (p2 + 1) * 4));
  w.tA = reinterpret_cast<float *>(take(V * heads * (p2 + 1) * 4));
  w.q = reinterpret_cast<float *>(take(D * 4));
  w.r = reinterpret_cast<float *>(take(heads * D * 4));
  w.Wt = reinterpret_cast<float *>(take(V * D * (p2 + 1) * 4));
  w.d_r = reinterpret_cast<float *>(take(heads * D * 4));
  w.d_q = reinterpret_cast<float *>(take(D * 4));
  w.total = off;
  return w;
}

// ------------------------------------------------------------------ the two ends, enqueued
static int head_bwd_impl(reslim_ctx *c, const char *fn, const float *x, const float *tokens, const float *d_y, float *d_tokens,
                         const reslim_grads *g, int batch, void *ws, hipStream_t st) {
  const HeadWs w = plan_head_ws(c, batch, ws);
  const int D = c->cfg.embed_dim, dt = c->cfg.dtype, C = c->cfg.out_vars;
  const int Mi = batch * c->N;
  const int64_t M = static_cast<int64_t>(batch) * c->n_h;
  const int sH = c->cfg.scale * c->cfg.H, sW = c->cfg.scale * c->cfg.W;
  const double es = static_cast<double>(act_size(c)), dMi = Mi, dD = D;
  const double fine = static_cast<double>(batch) * C * sH * sW;
  // transpose of un-patchify
  {
    const int64_t total = static_cast<int64_t>(Mi) * c->head_out;
    const dim3 grid(static_cast<unsigned>((total + 255) / 256));
    const int64_t total4 = static_cast<int64_t>(batch) * c->Hp * ((c->Wp + 3) / 4) * C * c->ps * 4 * (c->ps / 4);
    const dim3 grid4(static_cast<unsigned>((total4 + 255) / 256));
    const bool vec = c->ps % 4 == 0 && sW % 4 == 0 && (reinterpret_cast<uintptr_t>(d_y) & 15) == 0;
    if (dt == RESLIM_BF16 && vec)
      RESLIM_LAUNCH("patchify_grad", 0, 4.0 * fine + es * fine,
                    (patchify_act4_kernel<bf16_t><<<grid4, dim3(256), 0, st>>>(d_y, static_cast<bf16_t *>(w.dP), total4, c->Hp, c->Wp, C, c->ps, sH, sW), hipGetLastError()));
    else if (dt == RESLIM_BF16)
      RESLIM_LAUNCH("patchify_grad", 0, 4.0 * fine + es * fine,
                    (patchify_act_kernel<bf16_t><<<grid, dim3(256), 0, st>>>(d_y, static_cast<bf16_t *>(w.dP), total, c->N, c->Wp, C, c->ps, sH, sW), hipGetLastError()));
    else if (vec)
      RESLIM_LAUNCH("patchify_grad", 0, 8.0 * fine,
                    (patchify_act4_kernel<float><<<grid4, dim3(256), 0, st>>>(d_y, static_cast<float *>(w.dP), total4, c->Hp, c->Wp, C, c->ps, sH, sW), hipGetLastError()));
    else
      RESLIM_LAUNCH("patchify_grad", 0, 8.0 * fine,
                    (patchify_act_kernel<float><<<grid, dim3(256), 0, st>>>(d_y, static_cast<float *>(w.dP), total, c->N, c->Wp, C, c->ps, sH, sW), hipGetLastError()));
  }
  // residual path: weights and bias of the convolution
  {
    ResGradArgs a;
    a.x = x; a.dy = d_y; a.partial = w.resp; a.tiles = c->d_tiles; a.out_var_idx = c->d_out_var_idx;
    a.V = c->cfg.in_vars; a.C = C; a.H = c->cfg.H; a.W = c->cfg.W; a.s = c->cfg.scale; a.p = c->cfg.patch; a.ps = c->ps;
    a.T = c->T; a.batch = batch;
    (void)residual_grid(c, batch, &a.nbx, &a.nby);
    a.cwh = 17 / a.s + 3;
    a.cww = 65 / a.s + 3;
    const int n_acc = 9 * C * C + C;
    // as many outputs per pass as fit beside the other arrays in 150 KB of LDS
    int co = C > 8 ? 16 : C > 4 ? 8 : 4;
    while (co > 4 && residual_wgrad_lds_floats(C, co, a.cwh, a.cww) * sizeof(float) > kResGradLds) co /= 2;
    const size_t lds = residual_wgrad_lds_floats(C, co, a.cwh, a.cww) * sizeof(float);
    if (lds > kResGradLds || C > 64)                      // 64: the kernel's table of input variable indices
      return set_error(c, RESLIM_ESHAPE, std::string(fn) + ": the residual-path gradient's arrays do not fit in LDS (scale too small or too many variables)");
    const double win = static_cast<double>(a.cwh) * a.cww * a.nbx * a.nby * c->T * batch;   // coarse-window pixels over all blocks
    const double res_flop = 2.0 * (12.0 * fine + 9.0 * (C + 2.0) * C * win);
    // columns per run of the column step: 4 NIT >= 2 s + 3 (a run is shorter than 2 s + 1, plus alignment)
    const int nit = a.s <= 4 ? 3 : a.s <= 8 ? 5 : 16;
    hipError_t le = hipSuccess;
#define RESLIM_RESGRAD(O, N) (residual_wgrad_kernel<O, N><<<dim3(w.res_wg), dim3(256), lds, st>>>(a), hipGetLastError())
    RESLIM_LAUNCH("residual_wgrad", res_flop, 4.0 * fine + 4.0 * batch * C * c->cfg.H * c->cfg.W,
                  (le = co == 16 ? (nit == 3 ? RESLIM_RESGRAD(4, 3) : nit == 5 ? RESLIM_RESGRAD(4, 5) : RESLIM_RESGRAD(4, 16))
                      : co == 8  ? (nit == 3 ? RESLIM_RESGRAD(2, 3) : nit == 5 ? RESLIM_RESGRAD(2, 5) : RESLIM_RESGRAD(2, 16))
                                 : (nit == 3 ? RESLIM_RESGRAD(1, 3) : nit == 5 ? RESLIM_RESGRAD(1, 5) : RESLIM_RESGRAD(1, 16)),
                   le));
#undef RESLIM_RESGRAD
    RESLIM_LAUNCH("partial_reduce", 0, 4.0 * w.res_wg * n_acc, launch_partial_reduce(w.resp, g->w_res, w.res_wg, n_acc, 9 * C * C, st));
    RESLIM_LAUNCH("partial_reduce", 0, 4.0 * w.res_wg * C, launch_partial_reduce(w.resp + 9 * C * C, g->b_res, w.res_wg, n_acc, C, st));
  }
  // head GEMM: the final LayerNorm's output on the interior tokens is recomputed, not kept
  RESLIM_LAUNCH("layernorm_final", 0, dMi * dD * (4.0 + es),
                launch_layernorm(dt, tokens, c->d_interior_src, c->N, c->n_h, c->d_lnf_g, c->d_lnf_b, w.Af, Mi, D, st));
  {
    const double dN = c->head_out, dK = D;
    RESLIM_LAUNCH("gemm_dgrad", 2.0 * dMi * dN * dK, dMi * dN * es + dN * dK * es + dMi * dK * es,
                  launch_gemm(dt, EPI_BIAS_ACT, w.dP, c->train.wt_head, c->d_zero_bias, w.dAf, D, nullptr, 0, Mi, D, c->head_out, st));
    const WgradOp op = {w.dP, w.Af, g->w_head, g->b_head, c->head_out, D};
    RESLIM_LAUNCH("gemm_wgrad", 2.0 * dMi * dN * dK, dMi * dN * es + dMi * dK * es + 4.0 * dN * dK, launch_wgrad(dt, &op, 1, Mi, w.wgrad, st));
  }
  // final LayerNorm backwards on the interior rows, then back into the tile-major stream (halo rows: zero)
  RESLIM_LAUNCH("gather", 0, 8.0 * dMi * dD, launch_gather_rows(tokens, c->d_interior_src, w.Xi, batch, c->N, static_cast<int>(c->n_h), D, st));
  RESLIM_LAUNCH("layernorm_bwd", 0, dMi * dD * (8.0 + es),
                launch_layernorm_bwd(dt, w.Xi, w.dAf, c->d_lnf_g, nullptr, w.dXi, nullptr, w.lnp, g->lnf_g, g->lnf_b, Mi, D, st));
  RESLIM_LAUNCH("scatter_interior", 0, 4.0 * dMi * dD + 4.0 * static_cast<double>(M) * dD,
                (scatter_interior_kernel<<<dim3(static_cast<unsigned>((M + 3) / 4)), dim3(256), 0, st>>>(
                     w.dXi, c->d_gather, c->d_interior_src, d_tokens, M, c->n_h, c->N, D),
                 hipGetLastError()));
  return RESLIM_OK;
}

static int embed_bwd_impl(reslim_ctx *c, const char *fn, const float *x, const float *d_tokens, const reslim_grads *g, int batch,
                          void *ws, hipStream_t st) {
  const EmbedWs w = plan_embed_ws(c, batch, ws);
  const TrainModel &tm = c->train;
  const int D = c->cfg.embed_dim, dt = c->cfg.dtype, V = c->cfg.in_vars, heads = c->cfg.heads, dh = c->dh;
  const int p = c->cfg.patch, p2 = p * p;
  const int Mi = batch * c->N;
  const double es = static_cast<double>(act_size(c)), dMi = Mi, dD = D;
  const float kappa = 1.0f / sqrtf(static_cast<float>(dh));
  // gather transposed
  {
    const dim3 grid(static_cast<unsigned>((Mi + 3) / 4));
    if (dt == RESLIM_BF16)
      RESLIM_LAUNCH("gather_grad", 0, 4.0 * batch * static_cast<double>(c->n_h) * dD + (4.0 + es) * dMi * dD,
                    (gather_transpose_kernel<bf16_t><<<grid, dim3(256), 0, st>>>(d_tokens, c->d_copy_off, c->d_copy_idx, w.dz, static_cast<bf16_t *>(w.dz_act), Mi, c->n_h, c->N, D), hipGetLastError()));
    else
      RESLIM_LAUNCH("gather_grad", 0, 4.0 * batch * static_cast<double>(c->n_h) * dD + 8.0 * dMi * dD,
                    (gather_transpose_kernel<float><<<grid, dim3(256), 0, st>>>(d_tokens, c->d_copy_off, c->d_copy_idx, w.dz, static_cast<float *>(w.dz_act), Mi, c->n_h, c->N, D), hipGetLastError()));
  }
  // position rows (shared by the samples), aggregated values again, output map of the aggregation
  {
    const int64_t n = static_cast<int64_t>(c->N) * D;
    RESLIM_LAUNCH("pos_grad", 0, 4.0 * dMi * dD + 4.0 * n,
                  (batch_sum_kernel<<<dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, st>>>(w.dz, g->pos_emb, n, n, batch), hipGetLastError()));
  }
  RESLIM_LAUNCH("embed_agg", 0, 4.0 * batch * V * c->cfg.H * c->cfg.W + dMi * dD * es, launch_embed_agg(c, x, w.o, batch, st));
  {
    RESLIM_LAUNCH("gemm_dgrad", 2.0 * dMi * dD * dD, 2.0 * dMi * dD * es + dD * dD * es,
                  launch_gemm(dt, EPI_BIAS_ACT, w.dz_act, tm.wt_agg_wo, c->d_zero_bias, w.d_o, D, nullptr, 0, Mi, D, D, st));
    const WgradOp op = {w.dz_act, w.o, g->agg_wo, g->agg_bo, D, D};
    RESLIM_LAUNCH("gemm_wgrad", 2.0 * dMi * dD * dD, 2.0 * dMi * dD * es + 4.0 * dD * dD, launch_wgrad(dt, &op, 1, Mi, w.wgrad, st));
  }
  // folded aggregation backwards: logits, then the tables
  AggBwdArgs e;
  e.x = x; e.A = c->d_agg_A; e.a0 = c->d_agg_a0; e.d_o = w.d_o; e.a_out = w.a; e.x_out = w.xt; e.partial = w.pA;
  e.V = V; e.H = c->cfg.H; e.W = c->cfg.W; e.p = p; e.Wp = c->Wp; e.N = c->N; e.D = D; e.heads = heads; e.dh = dh; e.BN = Mi;
  {
    const TrainModel &tmm = c->train;
    const double dNe = tmm.n_e;
    RESLIM_LAUNCH("gemm_agg_dvalues", 2.0 * dMi * dNe * dD, dMi * dD * es + dNe * dD * es + 4.0 * dMi * dNe,
                  launch_gemm(dt, EPI_BIAS_F32, w.d_o, tmm.w_vtab, tmm.zero_e, w.E, tmm.n_e, nullptr, 0, Mi, tmm.n_e, D, st));
    e.E = w.E; e.ne = tmm.n_e;
    if (p2 != 4 && p2 != 1 && p2 != 16) return set_error(c, RESLIM_ESHAPE, std::string(fn) + ": the aggregation gradient is built for patch sizes 1, 2 and 4");
    if (w.lds_a > 150 * 1024) return set_error(c, RESLIM_ESHAPE, std::string(fn) + ": too many variables x heads for the aggregation gradient");
    const dim3 grid(static_cast<unsigned>(w.slabs_a));
    const double fl = 2.0 * dMi * heads * V * (3.0 * p2 + 4.0);
    const double by = 4.0 * dMi * dNe + 4.0 * dMi * V * (heads + p2 + 1.0);
    hipError_t le = hipSuccess;
#define RESLIM_AGGS(P2_) (w.tp == 16 ? (agg_scores_bwd_kernel<16, P2_><<<grid, dim3(256), w.lds_a, st>>>(e), hipGetLastError()) \
                                     : (agg_scores_bwd_kernel<4, P2_><<<grid, dim3(256), w.lds_a, st>>>(e), hipGetLastError()))
    RESLIM_LAUNCH("agg_scores_bwd", fl, by, (le = p2 == 4 ? RESLIM_AGGS(4) : p2 == 1 ? RESLIM_AGGS(1) : RESLIM_AGGS(16), le));
#undef RESLIM_AGGS
    const int64_t nA = static_cast<int64_t>(V) * heads * (p2 + 1);
    RESLIM_LAUNCH("partial_reduce", 0, 4.0 * w.slabs_a * nA, launch_partial_reduce(w.pA, w.tA, w.slabs_a, nA, nA, st));
  }
  {
    const int chunks = (dh + 63) / 64, rows = V * (p2 + 1);
    const dim3 grid(w.slabs_u, heads * chunks, (rows + 32 * w.mb_u - 1) / (32 * w.mb_u));
    const double fl = 2.0 * dMi * V * dD * (p2 + 1), by = dMi * dD * es + 4.0 * dMi * V * (heads + p2 + 1.0);
    hipError_t le = hipSuccess;
#define RESLIM_AGGV(T_, MB_) (agg_values_bwd_kernel<T_, MB_><<<grid, dim3(256), 0, st>>>(e, w.pU, w.tok_u, chunks), hipGetLastError())
    RESLIM_LAUNCH("agg_values_bwd", fl, by,
                  (le = dt == RESLIM_BF16 ? (w.mb_u == 1 ? RESLIM_AGGV(bf16_t, 1) : w.mb_u == 2 ? RESLIM_AGGV(bf16_t, 2) : w.mb_u == 3 ? RESLIM_AGGV(bf16_t, 3) : RESLIM_AGGV(bf16_t, 4))
                                          : (w.mb_u == 1 ? RESLIM_AGGV(float, 1) : w.mb_u == 2 ? RESLIM_AGGV(float, 2) : w.mb_u == 3 ? RESLIM_AGGV(float, 3) : RESLIM_AGGV(float, 4)),
                   le));
#undef RESLIM_AGGV
    const int64_t nU = static_cast<int64_t>(rows) * D;
    RESLIM_LAUNCH("partial_reduce", 0, 4.0 * w.slabs_u * nU, launch_partial_reduce(w.pU, w.tU, w.slabs_u, nU, nU, st));
  }
  // ---- chain rule through the fold
  FoldArgs f;
  f.w_pe = tm.w_pe; f.b_pe = tm.b_pe; f.var_emb = tm.var_emb; f.q0 = tm.q0; f.wq = tm.wq; f.bq = tm.bq; f.wk = tm.wk; f.bk = tm.bk; f.wv = tm.wv;
  f.tU = w.tU; f.tA = w.tA; f.agg_bo_grad = g->agg_bo;
  f.q = w.q; f.r = w.r; f.Wt = w.Wt; f.d_r = w.d_r; f.d_q = w.d_q;
  f.g_w_pe = g->w_pe; f.g_b_pe = g->b_pe; f.g_var_emb = g->var_emb; f.g_wv = g->agg_wv; f.g_bv = g->agg_bv; f.g_wk = g->agg_wk; f.g_bk = g->agg_bk;
  f.g_wq = g->agg_wq; f.g_bq = g->agg_bq; f.g_q0 = g->agg_q0; f.g_res = g->res_emb;
  f.V = V; f.D = D; f.dh = dh; f.heads = heads; f.p2 = p2; f.n_res = c->cfg.n_res; f.res_idx = c->cfg.res_idx; f.kappa = kappa;
  {
    const int q_blocks = (D + 3) / 4, rows = V * (p2 + 1), cols = (D + 31) / 32;
    const int64_t rest = static_cast<int64_t>(rows) * D + D + static_cast<int64_t>(c->cfg.n_res) * D;
    fold_prepare_kernel<<<dim3(static_cast<unsigned>(q_blocks + (rest + 255) / 256)), dim3(256), 0, st>>>(f, q_blocks);
    RESLIM_TRY("fold", hipGetLastError());
    fold_query_kernel<<<dim3((D + 63) / 64, heads), dim3(256), 0, st>>>(f);
    RESLIM_TRY("fold", hipGetLastError());
    const int n1 = cols * cols, n2 = (rows + 31) / 32 * cols, n3 = (heads + 31) / 32 * cols;
    fold_products_kernel<<<dim3(n1 + n2 + n3), dim3(256), 0, st>>>(f, n1, n2, cols);
    RESLIM_TRY("fold", hipGetLastError());
    fold_key_bwd_kernel<<<dim3(D), dim3(256), 0, st>>>(f);
    RESLIM_TRY("fold", hipGetLastError());
    fold_q0_kernel<<<dim3((D + 63) / 64), dim3(1024), 0, st>>>(f);
    RESLIM_TRY("fold", hipGetLastError());
  }
  return RESLIM_OK;
}

}  // namespace reslim

using namespace reslim;

// ------------------------------------------------------------------ entry points
extern "C" int reslim_bayes_loss_bwd(const float *pred, const float *target, const float *lat_w, int32_t batch, int32_t vars,
                                     int32_t Hf, int32_t Wf, float tv_weight, float upstream, float *d_pred, void *hip_stream) {
  if (!pred || !target || !lat_w || !d_pred) return RESLIM_EINVAL;
  if (batch < 1 || vars < 1 || Hf < 1 || Wf < 1 || static_cast<int64_t>(batch) * vars > 65535 || Hf > 65535) return RESLIM_EINVAL;
  const double count = static_cast<double>(batch) * vars * Hf * Wf;
  const double norm = 4.0 + 4.0 / 1.4142135623730951;
  const float data_f = static_cast<float>(2.0 * upstream / count);
  const float tv_f = static_cast<float>(2.0 * static_cast<double>(upstream) * tv_weight / (norm * count));
  // Work-groups of whole waves over a row, as even as they go.  Eight rows a thread where that still gives every CU eight waves
  // (a row is read 1.25 times), two and then one below that: there the chain of rows is what takes the time 16 planes of 180 x 360, loss and
  // gradient: 18.9 us with eight rows, 17.7 with two.
  const int64_t quads = (static_cast<int64_t>(Wf) + 3) / 4, groups = (quads + 255) / 256;
  const dim3 block(static_cast<unsigned>(((quads + groups - 1) / groups + 63) / 64 * 64));
  const int64_t waves = (quads + 63) / 64 * batch * vars, enough = 2048;
#define RESLIM_LOSS_BWD(RB, EVEN)                                                                                             \
  bayes_loss_bwd_kernel<RB, EVEN><<<dim3(static_cast<unsigned>(groups), (Hf + RB - 1) / RB, batch * vars), block, 0,          \
                                    static_cast<hipStream_t>(hip_stream)>>>(pred, target, lat_w, d_pred, Hf, Wf, data_f, tv_f)
#define RESLIM_LOSS_BWD_ROWS(EVEN)                                       \
  do {                                                                   \
    if (waves * ((Hf + 7) / 8) >= enough) RESLIM_LOSS_BWD(8, EVEN);      \
    else if (waves * ((Hf + 1) / 2) >= enough) RESLIM_LOSS_BWD(2, EVEN); \
    else RESLIM_LOSS_BWD(1, EVEN);                                       \
  } while (0)
  if (Wf % 4 == 0) RESLIM_LOSS_BWD_ROWS(true);
  else RESLIM_LOSS_BWD_ROWS(false);
#undef RESLIM_LOSS_BWD_ROWS
#undef RESLIM_LOSS_BWD
  return hipGetLastError() == hipSuccess ? RESLIM_OK : RESLIM_EHIP;
}

static hipError_t train_model_init() {
  hipError_t e = hipSuccess;
  const int lim = 150 * 1024;
#define RESLIM_ATTR(K) if (e == hipSuccess) e = hipFuncSetAttribute(reinterpret_cast<const void *>(&K), hipFuncAttributeMaxDynamicSharedMemorySize, lim)
  RESLIM_ATTR((agg_scores_bwd_kernel<16, 1>));
  RESLIM_ATTR((agg_scores_bwd_kernel<16, 4>));
  RESLIM_ATTR((agg_scores_bwd_kernel<16, 16>));
  RESLIM_ATTR((agg_scores_bwd_kernel<4, 1>));
  RESLIM_ATTR((agg_scores_bwd_kernel<4, 4>));
  RESLIM_ATTR((agg_scores_bwd_kernel<4, 16>));
  RESLIM_ATTR((residual_wgrad_kernel<4, 3>));
  RESLIM_ATTR((residual_wgrad_kernel<4, 5>));
  RESLIM_ATTR((residual_wgrad_kernel<4, 16>));
  RESLIM_ATTR((residual_wgrad_kernel<2, 3>));
  RESLIM_ATTR((residual_wgrad_kernel<2, 5>));
  RESLIM_ATTR((residual_wgrad_kernel<2, 16>));
  RESLIM_ATTR((residual_wgrad_kernel<1, 3>));
  RESLIM_ATTR((residual_wgrad_kernel<1, 5>));
  RESLIM_ATTR((residual_wgrad_kernel<1, 16>));
#undef RESLIM_ATTR
  return e;
}

extern "C" int reslim_train_prepare_model(reslim_ctx *c, const reslim_weights *wts) {
  const char *fn = "reslim_train_prepare_model";
  if (!c) return RESLIM_EINVAL;
  if (!wts) return set_error(c, RESLIM_EINVAL, std::string(fn) + ": null weights");
  if (c->train.ready) return RESLIM_OK;
  RESLIM_TRY("kernel setup", train_model_init());
  const int D = c->cfg.embed_dim, V = c->cfg.in_vars, p2 = c->cfg.patch * c->cfg.patch, dt = c->cfg.dtype;
  if (dt == RESLIM_BF16 && c->head_out % 64 != 0)
    return set_error(c, RESLIM_ESHAPE, std::string(fn) + ": out_vars * (patch * scale)^2 must be a multiple of 64 on the bfloat16 path (contraction length of the head's input gradient)");
  if (D % 4 != 0) return set_error(c, RESLIM_ESHAPE, std::string(fn) + ": embed_dim must be a multiple of 4");
  int rc = reslim_train_prepare(c);
  if (rc != RESLIM_OK) return rc;
  TrainModel &tm = c->train;
  auto up = [&](const float *src, size_t n, float **dst) -> hipError_t {
    void *d = nullptr;
    hipError_t e = hipMalloc(&d, std::max<size_t>(n * sizeof(float), 256));
    if (e != hipSuccess) return e;
    c->allocs.push_back(d);
    *dst = static_cast<float *>(d);
    return hipMemcpy(d, src, n * sizeof(float), hipMemcpyHostToDevice);
  };
  const size_t DD = static_cast<size_t>(D) * D;
  hipError_t e = up(wts->w_pe, static_cast<size_t>(V) * D * p2, &tm.w_pe);
  if (e == hipSuccess) e = up(wts->b_pe, static_cast<size_t>(V) * D, &tm.b_pe);
  if (e == hipSuccess) e = up(wts->var_emb, static_cast<size_t>(V) * D, &tm.var_emb);
  if (e == hipSuccess) e = up(wts->agg_q0, D, &tm.q0);
  if (e == hipSuccess) e = up(wts->agg_wq, DD, &tm.wq);
  if (e == hipSuccess) e = up(wts->agg_bq, D, &tm.bq);
  if (e == hipSuccess) e = up(wts->agg_wk, DD, &tm.wk);
  if (e == hipSuccess) e = up(wts->agg_bk, D, &tm.bk);
  if (e == hipSuccess) e = up(wts->agg_wv, DD, &tm.wv);
  if (e == hipSuccess) e = up(wts->agg_bv, D, &tm.bv);
  // [in, out] copies of the head's and the aggregation's output maps for their input gradients
  const size_t es = act_size(c);
  auto transposed = [&](const void *src, int rows, int cols, void **dst) -> hipError_t {
    void *d = nullptr;
    hipError_t e2 = hipMalloc(&d, std::max<size_t>(static_cast<size_t>(rows) * cols * es, 256));
    if (e2 != hipSuccess) return e2;
    c->allocs.push_back(d);
    *dst = d;
    return launch_transpose(dt, src, d, rows, cols, nullptr);
  };
  if (e == hipSuccess) e = transposed(c->d_w_head, c->head_out, D, &tm.wt_head);
  if (e == hipSuccess) e = transposed(c->d_agg_wo, D, D, &tm.wt_agg_wo);
  // the value table by (head, variable, pixel | offset) for the GEMM of the aggregation gradient
  if (e == hipSuccess) {
    const int rows = c->cfg.heads * V * (p2 + 1);
    tm.n_e = agg_table_rows(c);
    void *dw = nullptr, *dz = nullptr;
    const size_t es = dt == RESLIM_BF16 ? 2 : 4;
    e = hipMalloc(&dw, static_cast<size_t>(tm.n_e) * D * es);
    if (e == hipSuccess) { c->allocs.push_back(dw); e = hipMalloc(&dz, static_cast<size_t>(tm.n_e) * 4); }
    if (e == hipSuccess) { c->allocs.push_back(dz); e = hipMemset(dz, 0, static_cast<size_t>(tm.n_e) * 4); }
    if (e == hipSuccess) {
      const dim3 grid(static_cast<unsigned>((static_cast<int64_t>(tm.n_e) * D + 255) / 256));
      if (dt == RESLIM_BF16)
        agg_value_table_kernel<bf16_t><<<grid, dim3(256)>>>(c->d_agg_U, c->d_agg_c, static_cast<bf16_t *>(dw), V, D, c->dh, p2, rows, tm.n_e);
      else
        agg_value_table_kernel<float><<<grid, dim3(256)>>>(c->d_agg_U, c->d_agg_c, static_cast<float *>(dw), V, D, c->dh, p2, rows, tm.n_e);
      e = hipGetLastError();
    }
    tm.w_vtab = dw;
    tm.zero_e = static_cast<float *>(dz);
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) return set_error(c, e == hipErrorOutOfMemory ? RESLIM_ENOMEM : RESLIM_EHIP, std::string(fn) + ": " + hipGetErrorString(e));
  tm.ready = true;
  return RESLIM_OK;
}

static bool grads_complete(const reslim_grads *g, int first, int last) {
  const float *const *p = reinterpret_cast<const float *const *>(g);
  for (int i = first; i < last; ++i)
    if (!p[i]) return false;
  return true;
}
// field ranges of reslim_grads: front end [0, 14), blocks [14, 26), back end [26, 32)
enum { G_FRONT0 = 0, G_BLOCK0 = 14, G_BACK0 = 26, G_END = 32 };

extern "C" int reslim_head_bwd_workspace_bytes(const reslim_ctx *c, int32_t batch, size_t *out) {
  if (!c || !out || batch < 1) return RESLIM_EINVAL;
  *out = plan_head_ws(c, batch, nullptr).total;
  return RESLIM_OK;
}
extern "C" int reslim_embed_bwd_workspace_bytes(const reslim_ctx *c, int32_t batch, size_t *out) {
  if (!c || !out || batch < 1) return RESLIM_EINVAL;
  *out = plan_embed_ws(c, batch, nullptr).total;
  return RESLIM_OK;
}

static int check_model_train(reslim_ctx *c, const char *fn, int batch, const void *ws, size_t ws_bytes, size_t need) {
  if (!c->train.ready) return set_error(c, RESLIM_EINVAL, std::string(fn) + ": call reslim_train_prepare_model first");
  int rc = check_common(c, fn, batch, nullptr, 0, false);
  if (rc != RESLIM_OK) return rc;
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255)) return set_error(c, RESLIM_EWORKSPACE, std::string(fn) + ": workspace null or not 256-byte aligned");
  if (ws_bytes < need) return set_error(c, RESLIM_EWORKSPACE, std::string(fn) + ": workspace too small");
  return RESLIM_OK;
}

extern "C" int reslim_head_bwd(reslim_ctx *c, const float *x, const float *tokens, const float *d_y, float *d_tokens,
                               const reslim_grads *grads, int32_t batch, void *workspace, size_t ws_bytes, void *hip_stream) {
  const char *fn = "reslim_head_bwd";
  if (!c) return RESLIM_EINVAL;
  if (!x || !tokens || !d_y || !d_tokens || !grads || !grads_complete(grads, G_BACK0, G_END))
    return set_error(c, RESLIM_EINVAL, std::string(fn) + ": null buffer");
  int rc = check_model_train(c, fn, batch, workspace, ws_bytes, plan_head_ws(c, batch, nullptr).total);
  if (rc != RESLIM_OK) return rc;
  return head_bwd_impl(c, fn, x, tokens, d_y, d_tokens, grads, batch, workspace, static_cast<hipStream_t>(hip_stream));
}

extern "C" int reslim_embed_bwd(reslim_ctx *c, const float *x, const float *d_tokens, const reslim_grads *grads, int32_t batch,
                                void *workspace, size_t ws_bytes, void *hip_stream) {
  const char *fn = "reslim_embed_bwd";
  if (!c) return RESLIM_EINVAL;
  if (!x || !d_tokens || !grads || !grads_complete(grads, G_FRONT0, G_BLOCK0))
    return set_error(c, RESLIM_EINVAL, std::string(fn) + ": null buffer");
  int rc = check_model_train(c, fn, batch, workspace, ws_bytes, plan_embed_ws(c, batch, nullptr).total);
  if (rc != RESLIM_OK) return rc;
  return embed_bwd_impl(c, fn, x, d_tokens, grads, batch, workspace, static_cast<hipStream_t>(hip_stream));
}

// ------------------------------------------------------------------ the whole step
namespace {
struct StepPlan {
  size_t stream_bytes;       // one [M, D] fp32 stream
  size_t block_saved;        // saved activations of one block
  size_t saved_total;        // (L + 1) streams + L block buffers
  size_t fwd_ws, block_ws, head_ws, embed_ws, loss_ws, dy_bytes;
  size_t ws_total;           // d_y | two gradient streams | max of the stage workspaces
};
StepPlan plan_step(const reslim_ctx *c, int batch) {
  StepPlan p;
  const size_t M = static_cast<size_t>(batch) * c->n_h, D = c->cfg.embed_dim;
  p.stream_bytes = align256(M * D * sizeof(float));
  size_t sb = 0, wb = 0;
  reslim_block_train_bytes(c, batch, &sb, &wb);
  p.block_saved = align256(sb);
  p.block_ws = wb;
  const size_t L = c->cfg.depth;
  p.saved_total = (L + 1) * p.stream_bytes + L * p.block_saved;
  p.fwd_ws = plan_workspace(c, batch, nullptr).total;
  p.head_ws = plan_head_ws(c, batch, nullptr).total;
  p.embed_ws = plan_embed_ws(c, batch, nullptr).total;
  size_t lw = 0;
  reslim_bayes_loss_workspace_bytes(batch, c->cfg.out_vars, c->cfg.scale * c->cfg.H, c->cfg.scale * c->cfg.W, &lw);
  p.loss_ws = align256(lw);
  p.dy_bytes = align256(static_cast<size_t>(batch) * c->cfg.out_vars * c->cfg.scale * c->cfg.H * c->cfg.scale * c->cfg.W * sizeof(float));
  const size_t stage = std::max(std::max(p.fwd_ws, p.block_ws), std::max(std::max(p.head_ws, p.embed_ws), p.loss_ws));
  p.ws_total = p.dy_bytes + 2 * p.stream_bytes + align256(stage);
  return p;
}
}  // namespace

extern "C" int reslim_train_step_bytes(const reslim_ctx *c, int32_t batch, size_t *saved_bytes, size_t *ws_bytes) {
  if (!c || batch < 1) return RESLIM_EINVAL;
  const StepPlan p = plan_step(c, batch);
  if (saved_bytes) *saved_bytes = p.saved_total;
  if (ws_bytes) *ws_bytes = p.ws_total;
  return RESLIM_OK;
}

extern "C" int reslim_train_step_grads(reslim_ctx *c, const float *x, const float *target, const float *lat_w, float tv_weight,
                                       float loss_scale, float *y, double *loss3, const reslim_grads *grads, int32_t batch,
                                       void *saved, size_t saved_bytes, void *workspace, size_t ws_bytes, void *hip_stream) {
  const char *fn = "reslim_train_step_grads";
  if (!c) return RESLIM_EINVAL;
  if (!x || !target || !lat_w || !y || !loss3 || !grads || !grads_complete(grads, G_FRONT0, G_END))
    return set_error(c, RESLIM_EINVAL, std::string(fn) + ": null buffer");
  if (!(loss_scale > 0.0f) || !std::isfinite(loss_scale)) return set_error(c, RESLIM_EINVAL, std::string(fn) + ": loss_scale must be positive and finite");
  if (reinterpret_cast<uintptr_t>(loss3) % 8) return set_error(c, RESLIM_EINVAL, std::string(fn) + ": loss3 must be 8-byte aligned");
  const StepPlan p = plan_step(c, batch);
  int rc = check_model_train(c, fn, batch, workspace, ws_bytes, p.ws_total);
  if (rc != RESLIM_OK) return rc;
  if (!saved || (reinterpret_cast<uintptr_t>(saved) & 255) || saved_bytes < p.saved_total)
    return set_error(c, RESLIM_EWORKSPACE, std::string(fn) + ": saved buffer null, misaligned or smaller than reslim_train_step_bytes()");
  hipStream_t st = static_cast<hipStream_t>(hip_stream);
  const int L = c->cfg.depth, C = c->cfg.out_vars, D = c->cfg.embed_dim;
  const int Hf = c->cfg.scale * c->cfg.H, Wf = c->cfg.scale * c->cfg.W;
  unsigned char *sv = static_cast<unsigned char *>(saved), *wsb = static_cast<unsigned char *>(workspace);
  auto stream = [&](int l) { return reinterpret_cast<float *>(sv + static_cast<size_t>(l) * p.stream_bytes); };
  auto bsaved = [&](int l) { return sv + static_cast<size_t>(L + 1) * p.stream_bytes + static_cast<size_t>(l) * p.block_saved; };
  float *d_y = reinterpret_cast<float *>(wsb);
  float *ga = reinterpret_cast<float *>(wsb + p.dy_bytes), *gb = reinterpret_cast<float *>(wsb + p.dy_bytes + p.stream_bytes);
  void *stage = wsb + p.dy_bytes + 2 * p.stream_bytes;
  const size_t stage_bytes = ws_bytes - (p.dy_bytes + 2 * p.stream_bytes);
  // ---- forward, keeping every block's input and intermediates
  if ((rc = reslim_embed_fwd(c, x, stream(0), batch, stage, stage_bytes, hip_stream)) != RESLIM_OK) return rc;
  for (int l = 0; l < L; ++l)
    if ((rc = reslim_block_fwd_train(c, l, stream(l), stream(l + 1), bsaved(l), p.block_saved, batch, stage, stage_bytes, hip_stream)) != RESLIM_OK) return rc;
  if ((rc = reslim_head_fwd(c, x, stream(L), y, batch, stage, stage_bytes, hip_stream)) != RESLIM_OK) return rc;
  // ---- loss value and its gradient (times the loss scale)
  if (reslim_bayes_loss_fwd(y, target, lat_w, batch, C, Hf, Wf, tv_weight, loss3, stage, stage_bytes, hip_stream) != RESLIM_OK)
    return set_error(c, RESLIM_EHIP, std::string(fn) + ": loss forward failed");
  if (reslim_bayes_loss_bwd(y, target, lat_w, batch, C, Hf, Wf, tv_weight, loss_scale, d_y, hip_stream) != RESLIM_OK)
    return set_error(c, RESLIM_EHIP, std::string(fn) + ": loss gradient failed");
  // ---- backward
  if ((rc = head_bwd_impl(c, fn, x, stream(L), d_y, ga, grads, batch, stage, st)) != RESLIM_OK) return rc;
  const size_t DD = static_cast<size_t>(D) * D, R = c->R;
  for (int l = L - 1; l >= 0; --l) {
    reslim_block_grads bg;
    bg.ln1_g = grads->ln1_g + static_cast<size_t>(l) * D; bg.ln1_b = grads->ln1_b + static_cast<size_t>(l) * D;
    bg.w_qkv = grads->w_qkv + l * 3 * DD; bg.b_qkv = grads->b_qkv + static_cast<size_t>(l) * 3 * D;
    bg.w_proj = grads->w_proj + l * DD; bg.b_proj = grads->b_proj + static_cast<size_t>(l) * D;
    bg.ln2_g = grads->ln2_g + static_cast<size_t>(l) * D; bg.ln2_b = grads->ln2_b + static_cast<size_t>(l) * D;
    bg.w_fc1 = grads->w_fc1 + l * R * D; bg.b_fc1 = grads->b_fc1 + l * R;
    bg.w_fc2 = grads->w_fc2 + l * R * D; bg.b_fc2 = grads->b_fc2 + static_cast<size_t>(l) * D;
    if ((rc = block_bwd_chained(c, l, stream(l), bsaved(l), p.block_saved, ga, gb, &bg, batch, stage, stage_bytes, hip_stream, l < L - 1, l > 0)) != RESLIM_OK) return rc;
    std::swap(ga, gb);
  }
  return embed_bwd_impl(c, fn, x, ga, grads, batch, stage, st);
}

extern "C" int reslim_grads_unscale(reslim_ctx *c, const reslim_grads *grads, float inv_scale, int32_t *found_inf, void *hip_stream) {
  const char *fn = "reslim_grads_unscale";
  if (!c) return RESLIM_EINVAL;
  if (!grads || !found_inf || !grads_complete(grads, G_FRONT0, G_END)) return set_error(c, RESLIM_EINVAL, std::string(fn) + ": null argument");
  if (!(inv_scale > 0.0f) || !std::isfinite(inv_scale)) return set_error(c, RESLIM_EINVAL, std::string(fn) + ": inv_scale must be positive and finite");
  const int64_t D = c->cfg.embed_dim, R = c->R, V = c->cfg.in_vars, L = c->cfg.depth, C = c->cfg.out_vars;
  const int64_t p2 = static_cast<int64_t>(c->cfg.patch) * c->cfg.patch;
  const int64_t sizes[32] = {V * D * p2, V * D, V * D, D, D * D, D, D * D, D, D * D, D, D * D, D, static_cast<int64_t>(c->N) * D, c->cfg.n_res * D,
                             L * D, L * D, L * 3 * D * D, L * 3 * D, L * D * D, L * D, L * D, L * D, L * R * D, L * R, L * D * R, L * D,
                             D, D, static_cast<int64_t>(c->head_out) * D, c->head_out, C * C * 9, C};
  float *const *ptrs = reinterpret_cast<float *const *>(grads);
  for (int i = 0; i < 32; i += 12) {
    const int n = std::min(12, 32 - i);
    RESLIM_TRY("launch", launch_unscale_check(const_cast<float **>(ptrs) + i, sizes + i, n, inv_scale, found_inf, static_cast<hipStream_t>(hip_stream)));
  }
  return RESLIM_OK;
}
