// Geometry of the attention kernels that take any window (na3d_any.hip): tiles
// of 16 tokens, the box of tokens on the other side that a tile reaches, and the
// walk over that box in chunks of 16.  Host and device code, no HIP runtime
// calls (a host test compiles it on its own).
#pragma once

#include <stdint.h>

namespace strata {
namespace any {

// Quotient by a fixed n >= 1 of any 0 <= i < 2^30: with 2^s < n <= 2^(s+1) and
// mul = floor(2^(32+s) / n) + 1 (one more at most where the division rounds up),
// mul n - 2^(32+s) < 2 n <= 2^(s+2), and i 2^(s+2) < 2^(32+s).
struct FastDiv {
  uint32_t n, mul, sh;
  __host__ __device__ explicit FastDiv(uint32_t d) : n(d), mul(0), sh(0) {
    if (d < 2) return;
    sh = 31 - __builtin_clz(d - 1);
    mul = (uint32_t)(4294967296.0 * (double)(1u << sh) / (double)d) + 1u;
  }
  __host__ __device__ __forceinline__ uint32_t div(uint32_t i) const {
    return n == 1 ? i : (uint32_t)(((uint64_t)i * mul) >> 32) >> sh;
  }
};

struct AnyDims {
  int heads, Z, H, W, kz, ky, kx;
  int lz, ly, lx;         // log2 extents of the 16-token tile
  FastDiv ty, tx;         // tiles along y and x
  FastDiv places;         // tiles of one grid
  uint32_t nbh;           // grids: batch * heads
  uint32_t blocks;        // workgroups
  int split;              // waves of a workgroup that share a tile's chunks (1, 2 or 4); the others take the
                          // same tile of the next 4 / split grids
  float scale;
  int norm;
  float eps;
};

// first position of the border-clamped window of position i
__host__ __device__ __forceinline__ int start(int i, int L, int k) {
  const int s = i - (k >> 1);
  return s < 0 ? 0 : s > L - k ? L - k : s;
}

// A tile and the box it walks (the same in every batch and head).
struct Walk {
  int z, y, x;      // the lane's token of the tile (column m), clamped into the grid
  bool live;        // that token lies inside the grid
  int oz, oy, ox;   // origin of the box
  int ny, nx;
  FastDiv dyx, dx;
  uint32_t n;       // tokens in the box
  int lz, ly, lx, cz, cy, cx;  // the lane's range inside the box: [l, l + c) per axis
  int H, W;

  // INV = false: the tile's tokens are queries, the box holds their windows;
  // INV = true: they are keys, the box holds the queries that see them.
  template <bool INV>
  static __host__ __device__ __forceinline__ void range(int i, int L, int k, int& lo, int& n) {
    if (!INV) {
      lo = start(i, L, k);
      n = k;
    } else {
      const int r = k >> 1;
      lo = i < k ? 0 : i - r;
      n = (i >= L - k ? L - 1 : i + r) - lo + 1;
    }
  }
  template <bool INV>
  static __host__ __device__ __forceinline__ int axis(int t, int lb, int L, int k, int m, int& pos, bool& in, int& o, int& l,
                                             int& c) {
    const int first = t << lb, last = min(first + (1 << lb), L) - 1;
    int lo0, n0, lo1, n1;
    range<INV>(first, L, k, lo0, n0);
    range<INV>(last, L, k, lo1, n1);
    o = lo0;
    pos = first + m;
    in = in && pos <= last;
    pos = min(pos, last);
    range<INV>(pos, L, k, l, c);
    l -= o;
    return lo1 + n1 - lo0;
  }
  template <bool INV>
  static __host__ __device__ __forceinline__ Walk make(const AnyDims& d, uint32_t tile, int m) {
    const uint32_t q0 = d.tx.div(tile), ix = tile - q0 * d.tx.n;
    const uint32_t iz = d.ty.div(q0), iy = q0 - iz * d.ty.n;
    int z, y, x, oz, oy, ox, lz, ly, lx, cz, cy, cx;
    bool live = true;
    const int nz = axis<INV>((int)iz, d.lz, d.Z, d.kz, m >> (d.lx + d.ly), z, live, oz, lz, cz);
    const int ny = axis<INV>((int)iy, d.ly, d.H, d.ky, (m >> d.lx) & ((1 << d.ly) - 1), y, live, oy, ly, cy);
    const int nx = axis<INV>((int)ix, d.lx, d.W, d.kx, m & ((1 << d.lx) - 1), x, live, ox, lx, cx);
    return Walk{z, y, x, live, oz, oy, ox, ny, nx,
                FastDiv((uint32_t)(ny * nx)), FastDiv((uint32_t)nx), (uint32_t)(nz * ny * nx),
                lz, ly, lx, cz, cy, cx, d.H, d.W};
  }
  __host__ __device__ __forceinline__ void at(uint32_t i, int& bz, int& by, int& bx) const {
    const uint32_t q = dyx.div(i), r = i - q * dyx.n, s = dx.div(r);
    bz = (int)q;
    by = (int)s;
    bx = (int)(r - s * dx.n);
  }
  // position in the (y, x) plane, and in the (z, y, x) grid, of a token of the box
  __host__ __device__ __forceinline__ uint32_t plane(int by, int bx) const {
    return (uint32_t)(oy + by) * (uint32_t)W + (uint32_t)(ox + bx);
  }
  __host__ __device__ __forceinline__ uint32_t tok(int bz, uint32_t p) const {
    return (uint32_t)(oz + bz) * ((uint32_t)H * (uint32_t)W) + p;
  }
  __host__ __device__ __forceinline__ uint32_t mine_in_plane() const { return (uint32_t)y * (uint32_t)W + (uint32_t)x; }
  __host__ __device__ __forceinline__ uint32_t mine() const { return (uint32_t)z * ((uint32_t)H * (uint32_t)W) + mine_in_plane(); }
  __host__ __device__ __forceinline__ bool sees(int bz, int by, int bx) const {
    return ((uint32_t)(bz - lz) < (uint32_t)cz) & ((uint32_t)(by - ly) < (uint32_t)cy) & ((uint32_t)(bx - lx) < (uint32_t)cx);
  }
  // bit r: token i + r of the box exists and the lane's token sees it
  __host__ __device__ __forceinline__ uint32_t four(uint32_t i) const {
    int bz, by, bx;
    at(min(i, n - 1), bz, by, bx);
    uint32_t bits = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      bits |= (uint32_t)((i + r < n) & sees(bz, by, bx)) << r;
      const bool ex = ++bx == nx;
      by += ex;
      bx = ex ? 0 : bx;
      const bool ey = by == ny;
      bz += ey;
      by = ey ? 0 : by;
    }
    return bits;
  }
};

// A run of chunks of the box, kept in LDS by the waves of a workgroup (they walk
// the same tile): grid position and plane position of every token (clamped into
// the box), and per chunk and lane (m, g) which of the chunk's tokens 4g + r the
// tile's token m sees.
constexpr int kRun = 32;
struct Run {
  uint32_t tok[16 * kRun], pl[16 * kRun];
  uint8_t see[64 * kRun];
};

// the part of thread tid of 256 (its lane is the walk's) in filling a run from token i0 of the box on
__host__ __device__ __forceinline__ void fill_run(const Walk& w, Run& t, uint32_t i0, int tid) {
  const uint32_t left = w.n - i0;
  for (uint32_t j = tid; j < 16 * kRun && j < ((left + 15) & ~15u); j += 256) {
    int bz, by, bx;
    w.at(min(i0 + j, w.n - 1), bz, by, bx);
    const uint32_t p = w.plane(by, bx);
    t.pl[j] = p;
    t.tok[j] = w.tok(bz, p);
  }
  for (uint32_t c = tid >> 6; c < kRun && 16 * c < left; c += 4)
    t.see[64 * c + (tid & 63)] = (uint8_t)w.four(i0 + 16 * c + 4 * ((tid & 63) >> 4));
}

// Tokens that a block of b positions of an axis reaches, at most
inline int box_extent(int b, int L, int k) { return L < b + k - 1 ? L : b + k - 1; }

// workgroups of a problem: every tile of a grid for one group of grids, then the next group
inline int64_t any_blocks(const AnyDims& d) {
  const int64_t per = 4 / d.split;
  return ((int64_t)d.nbh + per - 1) / per * d.places.n;
}

// The tile's shape: of the 15 ways to write 16 = bz by bx, the one that needs
// the fewest chunks over the whole grid (ragged edges included), the longest in
// x among equals (its loads are the most contiguous).  A plane window takes
// 1 x 4 x 4, a column window 16 x 1 x 1.
inline AnyDims any_dims(int B, int heads, int Z, int H, int W, int kz, int ky, int kx, float scale, int norm, float eps) {
  int best[3] = {0, 2, 2};
  int64_t cost = INT64_MAX, tiles = 0;
  for (int lx = 4; lx >= 0; --lx)
    for (int ly = 4 - lx; ly >= 0; --ly) {
      const int lz = 4 - lx - ly;
      auto count = [](int L, int l) { return ((int64_t)L + (1 << l) - 1) >> l; };
      const int64_t t = count(Z, lz) * count(H, ly) * count(W, lx);
      const int64_t n = (int64_t)box_extent(1 << lz, Z, kz) * box_extent(1 << ly, H, ky) * box_extent(1 << lx, W, kx);
      const int64_t c = t * ((n + 15) / 16);
      if (c < cost) {
        cost = c;
        tiles = t;
        best[0] = lz; best[1] = ly; best[2] = lx;
      }
    }
  auto count = [](int L, int l) { return FastDiv((uint32_t)(((int64_t)L + (1 << l) - 1) >> l)); };
  const int64_t nbh = (int64_t)B * heads;
  // Fewer tiles than 4 waves per SIMD of the 256 CUs, or grids that do not fill
  // the workgroups' other waves (more than 15% of them idle): 2 or 4 waves share
  // a tile's chunks
  int split = tiles * nbh >= 4096 ? 1 : tiles * nbh >= 2048 ? 2 : 4;
  auto idle = [nbh](int per) { return (nbh + per - 1) / per * per * 20 > nbh * 23; };
  while (split < 4 && idle(4 / split)) split *= 2;
  AnyDims d{heads, Z, H, W, kz, ky, kx, best[0], best[1], best[2], count(H, best[1]), count(W, best[2]),
            FastDiv((uint32_t)tiles), (uint32_t)nbh, 0, split, scale, norm, eps};
  d.blocks = (uint32_t)any_blocks(d);
  return d;
}

// The launch grid of n workgroups.  A dimension of it holds fewer than 2^32
// threads, so of 256-thread workgroups at most 2^24 - 1: more than 2^23 go into
// rows of 2^23, and those of the last row past the n-th do nothing.
struct LaunchGrid {
  uint32_t x, y;
};
inline LaunchGrid launch_grid(int64_t n) {
  const int64_t row = (int64_t)1 << 23;
  return n <= row ? LaunchGrid{(uint32_t)n, 1} : LaunchGrid{(uint32_t)row, (uint32_t)((n + row - 1) / row)};
}

// The place in the problem of the i-th workgroup launched, of n.  Consecutive
// places stay on one XCD (workgroups are handed to the eight XCDs in turn): they
// share most of their box.
__host__ __device__ __forceinline__ uint32_t xcd_order(uint32_t i, uint32_t n) {
  const uint32_t q = n / 8, r = n % 8, x = i % 8;
  return x * q + min(x, r) + i / 8;
}

// Positions of an axis that a tile's box spans, at most: the queries that see keys
// i .. i + 15 are those from 0 on where i < k and those up to L - 1 where i + 15 >=
// L - k, so all of them on an axis of up to 2 k + 14.
inline int64_t box_most(int64_t L, int64_t k) { return L < 16 + 2 * k ? L : 16 + 2 * k; }

// Whether the 32-bit token and block indices above hold: every problem that a
// device can hold (2^32 tokens of the narrowest rows are 256 GiB a tensor) and
// whose windows can be walked in a lifetime.
inline bool any_fits(int B, int heads, int Z, int H, int W, int kz, int ky, int kx) {
  return (double)B * heads * Z * H * W < 4294967296.0 &&
         (double)box_most(Z, kz) * (double)box_most(H, ky) * (double)box_most(W, kx) < 1073741824.0 &&
         any_blocks(any_dims(B, heads, Z, H, W, kz, ky, kx, 1.f, 0, 0.f)) < ((int64_t)1 << 30);
}

}  // namespace any
}  // namespace strata
