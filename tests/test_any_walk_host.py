"""Host check of the tile geometry of the any-window attention kernels
(`csrc/any_walk.h`), compiled with g++ on its own.

For grids and windows of every form (odd windows, windows that span their axis
with either parity, columns, single positions, extents that the tile does not
divide): the tiles' live tokens cover the grid once; the chunks of every tile
stay inside the grid and show each lane exactly the tokens of its
border-clamped window (Sec. 3.2), or the queries whose window holds it, once
each, by brute force over the definition; every (batch, head) gets a wave; and
the division by a fixed number is exact up to 2^30.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2606_31248_amd", "csrc")

HARNESS = r"""
#define __host__
#define __device__
#define __forceinline__ inline
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>
using std::max;
using std::min;
#include "any_walk.h"
using namespace strata::any;

static int begin_of(int q, int L, int k) {  // nearest window of k positions inside [0, L)
  int s = q - (k - 1) / 2;
  return s < 0 ? 0 : s + k > L ? L - k : s;
}
static bool holds(int q, int j, int L, int k) { const int s = begin_of(q, L, k); return j >= s && j < s + k; }

template <bool INV>
static int check(int B, int heads, int Z, int H, int W, int kz, int ky, int kx) {
  const AnyDims d = any_dims(B, heads, Z, H, W, kz, ky, kx, 1.f, 0, 0.f);
  const int N = Z * H * W, per = 4 / d.split;
  if (d.nbh != (uint32_t)(B * heads) || (int64_t)d.blocks != any_blocks(d) || any_blocks(d) != (int64_t)d.places.n * ((B * heads + per - 1) / per)) return printf("blocks\n"), 1;
  std::vector<int> cover(N, 0);
  static Run run;
  for (uint32_t t = 0; t < d.places.n; ++t) {
    std::vector<Walk> w;
    for (int m = 0; m < 16; ++m) {
      w.push_back(Walk::make<INV>(d, t, m));
      const Walk& a = w.back();
      if (a.z < 0 || a.z >= Z || a.y < 0 || a.y >= H || a.x < 0 || a.x >= W) return printf("token outside\n"), 1;
      if (a.live) cover[a.mine()]++;
      if (a.mine() != (uint32_t)((a.z * H + a.y) * W + a.x) || a.n != w[0].n) return printf("tile\n"), 1;
    }
    if (t > 40 && t % 7) continue;  // the walk of a part of the tiles
    std::vector<int> seen(16 * N, 0);
    for (uint32_t i0 = 0; i0 < w[0].n; i0 += 16 * kRun) {
      for (int j = 0; j < 16 * kRun; ++j) run.tok[j] = run.pl[j] = ~0u;
      for (int tid = 0; tid < 256; ++tid) fill_run(w[tid & 15], run, i0, tid);
      for (uint32_t c = 0; c < min((uint32_t)kRun, (w[0].n - i0 + 15) / 16); ++c)
        for (int lane = 0; lane < 64; ++lane)
          for (int r = 0; r < 4; ++r) {
            const int j = 16 * c + 4 * (lane >> 4) + r;
            if (run.tok[j] >= (uint32_t)N || run.pl[j] != run.tok[j] % (uint32_t)(H * W)) return printf("token %u of %d\n", run.tok[j], N), 1;
            if (run.see[64 * c + lane] >> r & 1) seen[(lane & 15) * N + run.tok[j]]++;
          }
    }
    for (int m = 0; m < 16; ++m)
      for (int z = 0; z < Z; ++z)
        for (int y = 0; y < H; ++y)
          for (int x = 0; x < W; ++x) {
            const Walk& a = w[m];
            const bool want = INV ? holds(z, a.z, Z, kz) && holds(y, a.y, H, ky) && holds(x, a.x, W, kx)
                                  : holds(a.z, z, Z, kz) && holds(a.y, y, H, ky) && holds(a.x, x, W, kx);
            if (seen[m * N + (z * H + y) * W + x] != (want ? 1 : 0)) return printf("window of tile %d lane %d\n", (int)t, m), 1;
          }
  }
  for (int c : cover)
    if (c != 1) return printf("a token in %d tiles\n", c), 1;
  return 0;
}

int main() {
  std::mt19937 rng(7);
  auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
  for (int it = 0; it < 400; ++it) {
    int L[3], k[3];
    for (int a = 0; a < 3; ++a) {
      L[a] = pick(1, a == 0 ? 20 : 24);
      const int kind = pick(0, 4);
      k[a] = kind == 0 ? L[a] : kind == 1 ? 1 : min(2 * pick(0, 5) + 1, L[a] - (L[a] + 1) % 2);
      if (k[a] < 1) k[a] = 1;
    }
    const int B = pick(1, 2), h = pick(1, 3);
    if (check<false>(B, h, L[0], L[1], L[2], k[0], k[1], k[2]) || check<true>(B, h, L[0], L[1], L[2], k[0], k[1], k[2])) {
      printf("grid %dx%dx%d window %dx%dx%d\n", L[0], L[1], L[2], k[0], k[1], k[2]);
      return 1;
    }
  }
  for (int it = 0; it < 200000; ++it) {
    const uint32_t n = it < 4096 ? it + 1 : 1 + (uint32_t)(rng() % (1u << pick(1, 30)));
    const FastDiv f(n);
    const uint32_t q = ((1u << 30) - 1) / n;
    for (uint32_t i : {0u, n - 1, n, (uint32_t)(rng() >> 2), q * n - 1, q * n, (1u << 30) - 1})
      if (i < (1u << 30) && f.div(i) != i / n) return printf("%u / %u = %u\n", i, n, f.div(i)), 1;
  }
  // a tile's box along an axis, at every length up to 100 with every window: inside the axis, at most box_most long
  for (int L = 1; L <= 100; ++L)
    for (int k = 1; k <= L; ++k) {
      if (k % 2 == 0 && k < L) continue;
      for (int lb = 0; lb <= 4; ++lb)
        for (int t = 0; t << lb < L; ++t)
          for (int inv = 0; inv < 2; ++inv) {
            int pos, o, l, c;
            bool in = true;
            const int n = inv ? Walk::axis<true>(t, lb, L, k, 0, pos, in, o, l, c) : Walk::axis<false>(t, lb, L, k, 0, pos, in, o, l, c);
            if (o < 0 || o + n > L || n > box_most(L, k)) return printf("box of %d of %d, window %d\n", n, L, k), 1;
          }
    }
  for (int bh = 1; bh < 400; ++bh) {  // every grid has a wave, few waves have none
    const AnyDims d = any_dims(1, bh, 5, 9, 9, 3, 3, 3, 1.f, 0, 0.f);
    const int per = 4 / d.split, groups = (bh + per - 1) / per;
    if (groups * per < bh || groups * per > bh * 1.15 + 1e-9) return printf("%d grids: %d x %d\n", bh, groups, per), 1;
  }
  // launch grids: under 2^32 threads a dimension, every workgroup of the problem launched, and by any number
  // of launched ones every place taken once
  for (int64_t n : {(int64_t)1, (int64_t)8191, ((int64_t)1 << 24) - 1, (int64_t)1 << 24, ((int64_t)1 << 24) + 4, ((int64_t)1 << 30) - 1}) {
    const LaunchGrid g = launch_grid(n);
    if ((uint64_t)g.x * 256 >= 1ull << 32 || g.y > 65535 || (int64_t)g.x * g.y < n || (g.y > 1 && g.x % 8)) return printf("launch of %lld\n", (long long)n), 1;
    if (g.y == 1 && (int64_t)g.x != n) return printf("idle workgroups\n"), 1;
  }
  for (uint32_t n = 1; n < 600; ++n) {
    std::vector<int> seen(n, 0);
    for (uint32_t i = 0; i < n; ++i) {
      const uint32_t at = xcd_order(i, n);
      if (at >= n || seen[at]++) return printf("order of %u\n", n), 1;
    }
  }
  // 24 x 3345 x 3345 tokens of one (batch, head), 2^26 grids of one token: both hold, both need more than 2^24 workgroups
  for (const AnyDims& d : {any_dims(1, 1, 24, 3345, 3345, 3, 3, 3, 1.f, 0, 0.f), any_dims(1 << 22, 17, 1, 1, 1, 1, 1, 1, 1.f, 0, 0.f)})
    if (d.blocks < 1u << 24 || (int64_t)d.blocks != any_blocks(d) || (uint64_t)launch_grid(d.blocks).x * 256 >= 1ull << 32) return printf("large\n"), 1;
  if (!any_fits(1, 1, 24, 3345, 3345, 3, 3, 3) || !any_fits(1 << 22, 17, 1, 1, 1, 1, 1, 1)) return printf("large fits\n"), 1;
  if (any_fits(1, 1, 1 << 12, 1 << 12, 1 << 12, 3, 3, 3) || !any_fits(81, 16, 24, 128, 128, 9, 9, 9) || !any_fits(1 << 13, 1 << 13, 1, 1, 1, 1, 1, 1)) return printf("fits\n"), 1;
  printf("ok\n");
  return 0;
}
"""


def test_any_walk(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    src = tmp_path / "any_walk_check.cpp"
    exe = tmp_path / "any_walk_check"
    src.write_text(HARNESS)
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wall", "-Wno-unknown-pragmas", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok")


def test_waves_per_tile_of_the_gpu_shapes(tmp_path):
    """The number of waves that share a tile at each shape of the any-window GPU test is the one written there."""
    from test_gpu_any_window import SHAPES
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    assert {s[3] for s in SHAPES} == {1, 2, 4}
    src = tmp_path / "waves.cpp"
    exe = tmp_path / "waves"
    calls = "\n".join('printf("%d ", any_dims({}, 1.f, 0, 0.f).split);'.format(", ".join(map(str, s[0][:5] + s[1])))
                      for s in SHAPES)
    src.write_text(HARNESS[:HARNESS.index("int main()")] + "int main() {\n" + calls + "\nreturn 0;\n}\n")
    subprocess.run([gxx, "-O1", "-std=c++17", "-Wno-unused-function", "-Wno-unknown-pragmas", "-I", CSRC, str(src), "-o", str(exe)],
                   check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and [int(x) for x in out.stdout.split()] == [s[3] for s in SHAPES]
