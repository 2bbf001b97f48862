// Adaptive spatial compression, host side (ORBIT-2 Sec. 4.1, "Adaptive Spatial
// Compression"; Sec. 4.3 has the CPUs build the quad-trees while the GPUs compute):
// image -> 8-bit -> Canny edge map -> quad-tree on edge density -> leaf table.
// Integers throughout, apart from the 8-bit quantisation and the density test,
// which are single float32 operations in a fixed order.  No HIP call.
//
// A user pays for this on every batch of fields before the GPU can start, so every
// step is a loop over whole rows that the compiler turns into vector code: borders
// are padded in memory instead of clamped per pixel, values are as narrow as their
// range allows (8-bit image and classes, 16-bit filters), the division by 159 is an
// exact multiplication, the direction cases are selected instead of branched over,
// and only pixels that a strong neighbour promotes enter the flood fill.  The
// quad-tree reads its counts from a pyramid (its nodes are aligned squares).
// Best of many calls one after the other: one 180 x 360 field 1.0 -> 0.07 ms, four 128 x 256 fields in 64 haloed boxes
// 2.7 -> 0.33.  Between the other work of a program, whose data fills the caches, 0.12 and 0.42 with the binding; 0.6 to 0.9 ms
// on the first call.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <vector>

#include "reslim.h"

namespace {

#pragma clang fp contract(off)

// the box loops are compiled for the baseline and for 256-bit integers
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#define ASC_AVX2 __attribute__((target("avx2")))
#else
#define ASC_AVX2
#endif
#define ASC_INLINE inline __attribute__((always_inline))

constexpr int kPad = 2;       // columns on either side of a row: the 5 x 5 mask's reach
typedef int16_t v16 __attribute__((vector_size(32)));
typedef int32_t v16i __attribute__((vector_size(64)));
typedef uint8_t v16b __attribute__((vector_size(16)));
typedef float v8f __attribute__((vector_size(32)));
typedef int32_t v8i __attribute__((vector_size(32)));
typedef uint8_t v8b __attribute__((vector_size(8)));
ASC_INLINE v16 load16(const int16_t *p) {
  v16 v;
  std::memcpy(&v, p, 32);
  return v;
}

// Row buffers of one box, reused from box to box.  All maps share one pitch.
struct Maps {
  int H = 0, W = 0, pitch = 0;
  std::vector<uint8_t> q, cls, edge;       // image; 0 no candidate / 1 weak / 2 strong, one zero row above and below; edge pixels
  std::vector<int16_t> sm, gx, gy, mag;    // smoothed image, derivatives, magnitude (one zero row above and below)
  std::vector<uint16_t> ra, rb;            // outer and inner row pairs of the 5 x 5 mask
  std::vector<size_t> stack;
  void shape(int h, int w) {
    H = h;
    W = w;
    pitch = (w + 2 * kPad + 15) / 16 * 16 + 16;               // 16 columns past the row may be read and written
    const size_t n = static_cast<size_t>(h) * pitch, n2 = n + 2 * static_cast<size_t>(pitch);
    if (q.size() < n) {
      q.resize(n); sm.resize(n); gx.resize(n); gy.resize(n);
      mag.resize(n2); cls.resize(n2); edge.resize(n2);
    }
    if (ra.size() < static_cast<size_t>(pitch)) { ra.resize(pitch); rb.resize(pitch); }
  }
  size_t row(int y) const { return static_cast<size_t>(y) * pitch + kPad; }                    // maps without border rows
  size_t brow(int y) const { return static_cast<size_t>(y + 1) * pitch + kPad; }               // maps with them
};

// v -> floor((v - min) * (255 / (max - min)) + 0.5), clamped; a constant field maps to 0.  False: a pixel is not finite.
ASC_INLINE bool quantise(const float *v, size_t stride, Maps &m) {
  // finite floats in the order of their values as integers: integer minima and maxima become vector code
  int32_t mn = INT32_MAX, mx = INT32_MIN, worst = 0;        // worst: largest exponent-and-mantissa pattern
  for (int y = 0; y < m.H; ++y) {
    const float *r = v + y * stride;
    for (int x = 0; x < m.W; ++x) {
      int32_t i;
      std::memcpy(&i, r + x, 4);
      const int32_t mag = i & 0x7fffffff, key = i < 0 ? -mag : mag;
      mn = key < mn ? key : mn;
      mx = key > mx ? key : mx;
      worst = mag > worst ? mag : worst;
    }
  }
  if (worst >= 0x7f800000) return false;
  auto value = [](int32_t key) {
    const uint32_t bits = key < 0 ? 0x80000000u | static_cast<uint32_t>(-key) : static_cast<uint32_t>(key);
    float f;
    std::memcpy(&f, &bits, 4);
    return f;
  };
  const float lo = value(mn), hi = value(mx);
  const bool flat = !(hi > lo);
  const float scale = flat ? 0.0f : 255.0f / (hi - lo);
  for (int y = 0; y < m.H; ++y) {
    const float *__restrict r = v + y * stride;
    uint8_t *__restrict o = m.q.data() + m.row(y);
    if (flat) {
      std::memset(o - kPad, 0, m.pitch);
      continue;
    }
    auto pixels = [&](v8f f) {
      const v8f d = f - lo;
      const v8f p = d * scale;
      v8f t = p + 0.5f;
      t = t > 0.0f ? t : v8f{};              // also what a NaN of 0 * inf becomes; truncation is the floor from here on
      t = t < 255.0f ? t : v8f{} + 255.0f;
      return __builtin_convertvector(__builtin_convertvector(t, v8i), v8b);
    };
    int x = 0;
    for (; x + 8 <= m.W; x += 8) {
      v8f f;
      std::memcpy(&f, r + x, 32);
      const v8b b = pixels(f);
      std::memcpy(o + x, &b, 8);
    }
    if (x < m.W) {
      v8f f{};
      std::memcpy(&f, r + x, (m.W - x) * sizeof(float));
      const v8b b = pixels(f);
      std::memcpy(o + x, &b, 8);
    }
    for (int k = 1; k <= kPad; ++k) {
      o[-k] = o[0];
      o[m.W - 1 + k] = o[m.W - 1];
    }
  }
  return true;
}

// Canny's steps on the 8-bit image; edge[brow(y) + x] = 1 where an edge pixel is found
ASC_INLINE void canny(Maps &m, int low, int high) {
  const int H = m.H, W = m.W, P = m.pitch;
  auto clamp_row = [&](int y) { return std::min(std::max(y, 0), H - 1); };
  // 5 x 5 mask {2 4 5 4 2; 4 9 12 9 4; 5 12 15 12 5; ...} / 159 with rounding: rows y +- 2 and y +- 1 are added first
  for (int y = 0; y < H; ++y) {
    const uint8_t *c = m.q.data() + m.row(y);
    const uint8_t *u2 = m.q.data() + m.row(clamp_row(y - 2)), *d2 = m.q.data() + m.row(clamp_row(y + 2));
    const uint8_t *u1 = m.q.data() + m.row(clamp_row(y - 1)), *d1 = m.q.data() + m.row(clamp_row(y + 1));
    uint16_t *__restrict a = m.ra.data() + kPad, *__restrict b = m.rb.data() + kPad;
    for (int x = -kPad; x < W + kPad; ++x) {
      a[x] = static_cast<uint16_t>(u2[x] + d2[x]);
      b[x] = static_cast<uint16_t>(u1[x] + d1[x]);
    }
    int16_t *__restrict o = m.sm.data() + m.row(y);
    for (int x = 0; x < W; ++x) {
      const uint16_t a2 = a[x - 2] + a[x + 2], a1 = a[x - 1] + a[x + 1], b2 = b[x - 2] + b[x + 2], b1 = b[x - 1] + b[x + 1];
      const uint16_t c2 = static_cast<uint16_t>(c[x - 2] + c[x + 2]), c1 = static_cast<uint16_t>(c[x - 1] + c[x + 1]);
      const uint16_t t4 = a1 + b2, t5 = static_cast<uint16_t>(a[x] + c2), t12 = static_cast<uint16_t>(b[x] + c1);
      const uint16_t n = static_cast<uint16_t>(2 * a2 + 4 * t4 + 5 * t5 + 9 * b1 + 12 * t12 + 15 * c[x] + 79);       // <= 159 * 255 + 79
      // n / 159 for every n < 65,536: 52759 * 159 = 2^23 + 73 and 73 * 65,535 < 2^23
      o[x] = static_cast<int16_t>(static_cast<uint16_t>((static_cast<uint32_t>(n) * 52759u) >> 16) >> 7);
    }
    o[-1] = o[0];
    o[W] = o[W - 1];
  }
  for (int y = 0; y < H; ++y) {
    const int16_t *u = m.sm.data() + m.row(clamp_row(y - 1)), *c = m.sm.data() + m.row(y), *d = m.sm.data() + m.row(clamp_row(y + 1));
    int16_t *__restrict gx = m.gx.data() + m.row(y), *__restrict gy = m.gy.data() + m.row(y), *__restrict g = m.mag.data() + m.brow(y);
    for (int x = 0; x < W; ++x) {
      const int16_t l = static_cast<int16_t>(u[x - 1] + d[x - 1]), r = static_cast<int16_t>(u[x + 1] + d[x + 1]);
      const int16_t vx = static_cast<int16_t>(r + 2 * c[x + 1] - l - 2 * c[x - 1]);
      const int16_t vy = static_cast<int16_t>((d[x - 1] + 2 * d[x] + d[x + 1]) - (u[x - 1] + 2 * u[x] + u[x + 1]));
      gx[x] = vx;
      gy[x] = vy;
      g[x] = static_cast<int16_t>((vx < 0 ? -vx : vx) + (vy < 0 ? -vy : vy));
    }
    g[-1] = 0;
    g[W] = 0;
  }
  std::memset(m.mag.data(), 0, sizeof(int16_t) * P);
  std::memset(m.mag.data() + m.brow(H) - kPad, 0, sizeof(int16_t) * P);
  // suppression: the neighbours along the gradient are selected by direction sector, magnitude 0 outside the image
  const v16 lowv = v16{} + static_cast<int16_t>(std::min(low, 32767)), highv = v16{} + static_cast<int16_t>(std::min(high, 32767));
  constexpr int32_t kTan22 = 13573;   // tan(22.5 deg) in 15 fraction bits; tan(67.5 deg) = tan(22.5 deg) + 2
  std::memset(m.cls.data(), 0, P);
  std::memset(m.cls.data() + m.brow(H) - kPad, 0, P);
  for (int y = 0; y < H; ++y) {
    const int16_t *gx = m.gx.data() + m.row(y), *gy = m.gy.data() + m.row(y);
    const int16_t *c = m.mag.data() + m.brow(y), *u = c - P, *d = c + P;
    uint8_t *__restrict o = m.cls.data() + m.brow(y);
    // 16 pixels at a time.  With h = ax * kTan22 >> 15 (kTan22 is odd and ax < 2^15, so the product is a multiple of
    // 2^15 for ax = 0 alone): ay * 2^15 < ax * kTan22 is ay <= h and ax > 0; ay * 2^15 > ax * (kTan22 + 2^16) is
    // ay - 2 ax > h.  All values fit 16 bits (ax, ay <= 1020).
    for (int x = 0; x < W; x += 16) {
      const v16 vx = load16(gx + x), vy = load16(gy + x), v = load16(c + x);
      const v16 ax = vx < 0 ? -vx : vx, ay = vy < 0 ? -vy : vy;
      const v16 h = __builtin_convertvector((__builtin_convertvector(ax, v16i) * kTan22) >> 15, v16);
      const v16 across = (ay <= h) & (ax > 0), along = (ay - ax - ax) > h, same = (vx ^ vy) >= 0;
      const v16 before = across ? load16(c + x - 1) : along ? load16(u + x) : same ? load16(u + x - 1) : load16(u + x + 1);
      const v16 after = across ? load16(c + x + 1) : along ? load16(d + x) : same ? load16(d + x + 1) : load16(d + x - 1);
      const v16 keep = (v > lowv) & (v > before) & (v >= after);
      const v16 cls = -(keep + (keep & (v > highv)));
      const v16b bytes = __builtin_convertvector(cls, v16b);
      std::memcpy(o + x, &bytes, 16);
    }
    o[-1] = 0;
    o[W] = 0;
  }
  // hysteresis: strong pixels, weak pixels with a strong neighbour, then a flood from those through weak ones
  std::memset(m.edge.data(), 0, P);
  std::memset(m.edge.data() + m.brow(H) - kPad, 0, P);
  m.stack.clear();
  for (int y = 0; y < H; ++y) {
    const uint8_t *c = m.cls.data() + m.brow(y), *u = c - P, *d = c + P;
    uint8_t *__restrict o = m.edge.data() + m.brow(y);
    uint8_t any = 0;
    for (int x = 0; x < W; ++x) {
      const uint8_t around = static_cast<uint8_t>(u[x - 1] | u[x] | u[x + 1] | c[x - 1] | c[x + 1] | d[x - 1] | d[x] | d[x + 1]);
      const uint8_t strong = static_cast<uint8_t>(c[x] >> 1), promoted = static_cast<uint8_t>((c[x] & 1) & (around >> 1));
      o[x] = static_cast<uint8_t>(strong | (promoted << 1));            // 2: to be visited by the flood
      any |= promoted;
    }
    o[-1] = 0;
    o[W] = 0;
    if (!any) continue;
    for (int x0 = 0; x0 < W; x0 += 8) {
      uint64_t w;
      std::memcpy(&w, o + x0, 8);            // what lies past the row's end is not looked at below
      if (!(w & 0x0202020202020202u)) continue;
      for (int x = x0; x < x0 + 8 && x < W; ++x)
        if (o[x] & 2) {
          o[x] = 1;
          m.stack.push_back(m.brow(y) + x);
        }
    }
  }
  uint8_t *edge = m.edge.data();
  const uint8_t *cls = m.cls.data();
  const ptrdiff_t around[8] = {-P - 1, -P, -P + 1, -1, 1, P - 1, P, P + 1};
  while (!m.stack.empty()) {
    const size_t i = m.stack.back();
    m.stack.pop_back();
    for (ptrdiff_t s : around) {
      const size_t j = i + s;
      if (cls[j] && !edge[j]) {
        edge[j] = 1;
        m.stack.push_back(j);
      }
    }
  }
}

ASC_INLINE bool box_edges(const float *v, size_t stride, int low, int high, Maps &m) {
  if (!quantise(v, stride, m)) return false;
  canny(m, low, high);
  return true;
}
bool box_edges_base(const float *v, size_t stride, int low, int high, Maps &m) { return box_edges(v, stride, low, high, m); }
ASC_AVX2 bool box_edges_avx2(const float *v, size_t stride, int low, int high, Maps &m) { return box_edges(v, stride, low, high, m); }

// edge map of an H x W box whose rows are `stride` floats apart; false where a pixel is not finite
bool find_edges(const float *v, size_t stride, int H, int W, int low, int high, Maps &m) {
  m.shape(H, W);
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
  static const bool avx2 = __builtin_cpu_supports("avx2");
  if (avx2) return box_edges_avx2(v, stride, low, high, m);
#endif
  return box_edges_base(v, stride, low, high, m);
}

// Edge pixels of every aligned square of 1, 2, 4 .. max_leaf patches, as far as one fits into the grid (a node that
// sticks out splits without a look at its count), the grid padded with empty patches
struct Pyramid {
  std::vector<int32_t> n;
  std::vector<size_t> first;               // of every level
  int w0 = 0;                              // patches per row of level 0
  std::vector<uint16_t> col;
  void build(const Maps &m, int hp, int wp, int p, int max_leaf) {
    int most = 1;
    while (most < max_leaf && most <= std::min(hp, wp) / 2) most *= 2;
    const int hr = (hp + most - 1) / most * most;
    w0 = (wp + most - 1) / most * most;
    first.clear();
    size_t total = 0;
    for (int s = 1; s <= most; s *= 2) {
      first.push_back(total);
      total += static_cast<size_t>(hr / s) * (w0 / s);
    }
    n.assign(total, 0);
    col.resize(m.W);
    for (int py = 0; py < hp; ++py) {
      std::fill(col.begin(), col.end(), 0);
      for (int i = 0; i < p; ++i) {
        const uint8_t *e = m.edge.data() + m.brow(py * p + i);
        for (int x = 0; x < m.W; ++x) col[x] = static_cast<uint16_t>(col[x] + e[x]);
      }
      int32_t *o = n.data() + static_cast<size_t>(py) * w0;
      const uint16_t *c = col.data();
      if (p == 2) {
        for (int px = 0; px < wp; ++px) o[px] = c[2 * px] + c[2 * px + 1];
      } else {
        for (int px = 0; px < wp; ++px, c += p) {
          int32_t s = 0;
          for (int j = 0; j < p; ++j) s += c[j];
          o[px] = s;
        }
      }
    }
    for (size_t k = 1; k < first.size(); ++k) {
      const int w = w0 >> k, h = hr >> k;
      for (int y = 0; y < h; ++y) {
        const int32_t *a = n.data() + first[k - 1] + static_cast<size_t>(2 * y) * (2 * w), *b = a + 2 * w;
        int32_t *o = n.data() + first[k] + static_cast<size_t>(y) * w;
        for (int x = 0; x < w; ++x) o[x] = (a[2 * x] + a[2 * x + 1]) + (b[2 * x] + b[2 * x + 1]);
      }
    }
  }
  int32_t count(int level, int y0, int x0) const {
    return n[first[level] + static_cast<size_t>(y0 >> level) * (w0 >> level) + (x0 >> level)];
  }
};

struct TreeBuilder {
  const Pyramid &py;
  int Hp, Wp, p, min_leaf;
  float tau;
  int32_t *ly, *lx, *ls, *patch_leaf;
  int64_t n;                          // leaves written so far (batch-wide)

  void visit(int y0, int x0, int level) {
    if (y0 >= Hp || x0 >= Wp) return;                     // wholly in the padding of a ragged grid
    const int s = 1 << level;
    const bool inside = y0 + s <= Hp && x0 + s <= Wp;     // a node that sticks out always splits
    bool split = !inside;
    if (inside && s > min_leaf) {                         // only here is the area sure to fit: the node lies in the image
      const float area = static_cast<float>(static_cast<int64_t>(s) * p * s * p);
      const float bound = tau * area;
      split = static_cast<float>(py.count(level, y0, x0)) > bound;
    }
    if (split) {
      const int h = s / 2;
      visit(y0, x0, level - 1);
      visit(y0, x0 + h, level - 1);
      visit(y0 + h, x0, level - 1);
      visit(y0 + h, x0 + h, level - 1);
      return;
    }
    ly[n] = y0; lx[n] = x0; ls[n] = s;
    int32_t *o = patch_leaf + static_cast<size_t>(y0) * Wp + x0;
    const int32_t id = static_cast<int32_t>(n);
    for (int yy = 0; yy < s; ++yy, o += Wp)
      for (int xx = 0; xx < s; ++xx) o[xx] = id;
    ++n;
  }
  void grow(int max_leaf) {
    int top = 0;
    while ((1 << top) < max_leaf) ++top;
    for (int ry = 0; ry < Hp; ry += max_leaf)
      for (int rx = 0; rx < Wp; rx += max_leaf) visit(ry, rx, top);
  }
};

bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

}  // namespace

extern "C" int reslim_asc_build(const float *images, int32_t batch, int32_t H, int32_t W, int32_t patch, int32_t max_leaf,
                                int32_t min_leaf, int32_t canny_low, int32_t canny_high, float tau, int32_t *leaf_y0,
                                int32_t *leaf_x0, int32_t *leaf_s, int32_t *sample_off, int32_t *patch_leaf,
                                int64_t *n_leaves_out) {
  if (!images || !leaf_y0 || !leaf_x0 || !leaf_s || !sample_off || !patch_leaf || !n_leaves_out) return RESLIM_EINVAL;
  if (batch < 1 || H < 1 || W < 1 || patch < 1 || canny_low < 0 || canny_high < canny_low || !(tau >= 0.0f) || !std::isfinite(tau))
    return RESLIM_EINVAL;
  if (!pow2(max_leaf) || !pow2(min_leaf) || min_leaf > max_leaf || H % patch || W % patch) return RESLIM_ESHAPE;
  const int Hp = H / patch, Wp = W / patch;
  if (static_cast<int64_t>(batch) * Hp * Wp > INT32_MAX) return RESLIM_ESHAPE;
  const size_t npix = static_cast<size_t>(H) * W, N = static_cast<size_t>(Hp) * Wp;
  Maps m;
  Pyramid py;
  int64_t n = 0;
  sample_off[0] = 0;
  for (int b = 0; b < batch; ++b) {
    if (!find_edges(images + b * npix, W, H, W, canny_low, canny_high, m)) return RESLIM_EINVAL;
    py.build(m, Hp, Wp, patch, max_leaf);
    TreeBuilder tb{py, Hp, Wp, patch, min_leaf, tau, leaf_y0, leaf_x0, leaf_s, patch_leaf + b * N, n};
    tb.grow(max_leaf);
    n = tb.n;
    sample_off[b + 1] = static_cast<int32_t>(n);
  }
  *n_leaves_out = n;
  return RESLIM_OK;
}

// Compression combined with TILES: every (sample, tile) pair is compressed on its own, on the
// tile's haloed box of the field, exactly as reslim_asc_build treats a whole sample.
extern "C" int reslim_asc_build_tiles(const float *images, int32_t batch, int32_t H, int32_t W, int32_t patch,
                                      int32_t tiles_y, int32_t tiles_x, int32_t halo, int32_t max_leaf, int32_t min_leaf,
                                      int32_t canny_low, int32_t canny_high, float tau, int32_t *leaf_y0, int32_t *leaf_x0,
                                      int32_t *leaf_s, int32_t *seq_off, int32_t *patch_leaf, int64_t *n_leaves_out) {
  if (!images || !leaf_y0 || !leaf_x0 || !leaf_s || !seq_off || !patch_leaf || !n_leaves_out) return RESLIM_EINVAL;
  if (batch < 1 || H < 1 || W < 1 || patch < 1 || canny_low < 0 || canny_high < canny_low || !(tau >= 0.0f) || !std::isfinite(tau))
    return RESLIM_EINVAL;
  if (!pow2(max_leaf) || !pow2(min_leaf) || min_leaf > max_leaf || H % patch || W % patch) return RESLIM_ESHAPE;
  const int Hp = H / patch, Wp = W / patch;
  if (tiles_y < 1 || tiles_x < 1) return RESLIM_ESHAPE;
  const int T = tiles_y * tiles_x;
  std::vector<tile_desc> tiles(T);
  int64_t n_h = 0;
  const int rc = tiles_partition(Hp, Wp, tiles_y, tiles_x, halo, tiles.data(), nullptr, nullptr, &n_h);
  if (rc != RESLIM_OK) return rc;
  if (static_cast<int64_t>(batch) * n_h > INT32_MAX) return RESLIM_ESHAPE;
  const size_t npix = static_cast<size_t>(H) * W, N = static_cast<size_t>(Hp) * Wp;
  Maps m;
  Pyramid py;
  std::vector<int32_t> local;
  int64_t n = 0;
  seq_off[0] = 0;
  for (int b = 0; b < batch; ++b)
    for (int t = 0; t < T; ++t) {
      const tile_desc &td = tiles[t];
      const int hp = td.Y1 - td.Y0, wp = td.X1 - td.X0;
      const float *box = images + b * npix + static_cast<size_t>(td.Y0) * patch * W + static_cast<size_t>(td.X0) * patch;
      if (!find_edges(box, W, hp * patch, wp * patch, canny_low, canny_high, m)) return RESLIM_EINVAL;
      py.build(m, hp, wp, patch, max_leaf);
      local.resize(static_cast<size_t>(hp) * wp);
      const int64_t first = n;
      TreeBuilder tb{py, hp, wp, patch, min_leaf, tau, leaf_y0, leaf_x0, leaf_s, local.data(), n};
      tb.grow(max_leaf);
      n = tb.n;
      for (int64_t l = first; l < n; ++l) {          // box coordinates -> grid coordinates
        leaf_y0[l] += td.Y0;
        leaf_x0[l] += td.X0;
      }
      for (int yy = td.y0; yy < td.y1; ++yy)         // the tile's interior patches decompress from its own leaves
        std::copy_n(local.data() + static_cast<size_t>(yy - td.Y0) * wp + (td.x0 - td.X0), td.x1 - td.x0,
                    patch_leaf + b * N + static_cast<size_t>(yy) * Wp + td.x0);
      seq_off[static_cast<size_t>(b) * T + t + 1] = static_cast<int32_t>(n);
    }
  *n_leaves_out = n;
  return RESLIM_OK;
}

// Canny edge map of one 8-bit-quantised field, for inspection and tests: edges [H*W] 0/1
extern "C" int reslim_asc_edges(const float *image, int32_t H, int32_t W, int32_t canny_low, int32_t canny_high, uint8_t *edges_out) {
  if (!image || !edges_out || H < 1 || W < 1 || canny_low < 0 || canny_high < canny_low) return RESLIM_EINVAL;
  Maps m;
  if (!find_edges(image, W, H, W, canny_low, canny_high, m)) return RESLIM_EINVAL;
  for (int y = 0; y < H; ++y) std::memcpy(edges_out + static_cast<size_t>(y) * W, m.edge.data() + m.brow(y), W);
  return RESLIM_OK;
}
