// Neighbourhood attention for every problem without a 16-bit MFMA kernel: both
// dtypes, head_dim 32, 64 or 128, any window and grid.  All arithmetic is
// float32; the contractions run on the float32 matrix instruction
// v_mfma_f32_16x16x4_f32 (2048 FLOP per instruction, 154 TFLOP/s measured with
// a large matrix product), so nothing is rounded to 16 bits between the inputs
// and the results.
//
// A wave owns a tile of 16 tokens (queries in the forward and dq, keys in dk/dv)
// in a block of (z, y, x) extents whose product is 16, and walks the box of
// tokens on the other side that any of them sees, 16 at a time (a chunk), in
// linear order over the whole three-dimensional box, so that at most one chunk
// is padded.  What bounds it: the matrix instructions, 2 head_dim / 4 per chunk
// forward, 3 in dq, 4 in dk/dv, times the share of the box outside the windows.
//
// Layouts (lane l, m = l % 16, g = l / 16).  A 16 x 4 operand gives lane l row m,
// column g.  The sum over head_dim may take the channels in any order, so lane l
// holds the 16-byte pieces g, g + 4, ... of row m (whole pieces, one load each)
// and step s of the contraction takes element s of both operands.  The scores
// come out with the tile's token as the column m and the chunk's tokens 4g + r as
// the rows, which is the operand layout of the second product as it stands; its
// other operand holds, for token 4g + r, the head_dim / 16 channels from
// m head_dim / 16 on, so that output tile c, row m is channel m head_dim / 16 + c.
// In the backward the staged rows are needed in both layouts: the wave writes
// them to its own part of LDS and reads them back the other way.
//
// Measured against one thread per query (or one wave per query below 2^18) with
// float32 vector arithmetic: float32 forward and backward, 4 heads x 7x21x27,
// d 64, 5x9x9: 14733 -> 243 us; bf16 3x3x3 forward and backward, 6 tiles x 16
// heads x 24x16x16: 20589 -> 1180 us; float32 forward, 4 heads x 4x16x16, d 32,
// 3x7x7: 56.8 -> 13.6 us.
//
// Values outside a query's window never reach its results, infinities and NaN
// included: scores and weights are selected, and a chunk that holds a value that
// is not finite takes a scalar loop in which only the window's tokens are added
// (a product with a zero weight would spread it).
#include "common.h"

#include "any_walk.h"
#include "kernels.h"
#include "mfma_util.h"

namespace strata {
namespace {

using namespace any;
using mfma::f32x4;
using mfma::sum_over_rows;

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;
constexpr float kLowest = -3.402823466e38f;

template <typename T>
__device__ __forceinline__ float ldf(const T* p);
template <>
__device__ __forceinline__ float ldf<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ldf<uint16_t>(const uint16_t* p) { return bf16_to_f32(*p); }

// N consecutive values, N sizeof(T) a multiple of 4 and the address aligned to it (at most 16)
template <typename T, int N>
__device__ __forceinline__ void load_n(const T* p, float* f) {
  constexpr int W = N * (int)sizeof(T) / 4;
  uint32_t u[W];
  if constexpr (W % 4 == 0) {
#pragma unroll
    for (int i = 0; i < W; i += 4) {
      const uint4 a = *reinterpret_cast<const uint4*>(reinterpret_cast<const uint32_t*>(p) + i);
      u[i] = a.x; u[i + 1] = a.y; u[i + 2] = a.z; u[i + 3] = a.w;
    }
  } else if constexpr (W == 2) {
    const uint2 a = *reinterpret_cast<const uint2*>(p);
    u[0] = a.x; u[1] = a.y;
  } else {
    static_assert(W == 1, "");
    u[0] = *reinterpret_cast<const uint32_t*>(p);
  }
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] = __uint_as_float(u[i]);
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 2) {
      f[i] = __uint_as_float(u[i / 2] << 16);
      f[i + 1] = __uint_as_float(u[i / 2] & 0xFFFF0000u);
    }
  }
}

template <typename T, int N>
__device__ __forceinline__ void store_n(T* p, const float* f) {
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int i = 0; i < N; i += 4) *reinterpret_cast<float4*>(p + i) = make_float4(f[i], f[i + 1], f[i + 2], f[i + 3]);
  } else {
#pragma unroll
    for (int i = 0; i < N; i += 8)
      *reinterpret_cast<uint4*>(p + i) = make_uint4(pack_bf16x2(f[i], f[i + 1]), pack_bf16x2(f[i + 2], f[i + 3]),
                                                    pack_bf16x2(f[i + 4], f[i + 5]), pack_bf16x2(f[i + 6], f[i + 7]));
  }
}

// The lane's share of a row in the operand layout: pieces g, g + 4, ... of 16 bytes
template <typename T, int D>
struct Frag {
  static constexpr int E = 16 / (int)sizeof(T);  // elements of a piece
  static constexpr int NP = D / (4 * E);         // pieces per lane
  static constexpr int N = D / 4;                // elements per lane
  static __device__ __forceinline__ void load(const T* row, int g, float* f) {
#pragma unroll
    for (int j = 0; j < NP; ++j) load_n<T, E>(row + (4 * j + g) * E, f + j * E);
  }
  static __device__ __forceinline__ void rotate(const float2* ph, int g, float* f) {
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int e = 0; e < E; e += 4) {
        const float4 p = *reinterpret_cast<const float4*>(ph + ((4 * j + g) * E + e) / 2);
        float* x = f + j * E + e;
        const float a = x[0], b = x[1], c = x[2], d = x[3];
        x[0] = fmaf(a, p.x, -b * p.y);
        x[1] = fmaf(a, p.y, b * p.x);
        x[2] = fmaf(c, p.z, -d * p.w);
        x[3] = fmaf(c, p.w, d * p.z);
      }
  }
  // QK RMSNorm: divide the row (its four lanes together) by its root mean square
  static __device__ __forceinline__ void normalise(float* f, float eps) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) ss = fmaf(f[i], f[i], ss);
    const float r = 1.f / sqrtf(sum_over_rows(ss) / D + eps);
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] *= r;
  }
  static __device__ __forceinline__ void to_lds(float* row, int g, const float* f) {
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int e = 0; e < E; e += 4)
        *reinterpret_cast<float4*>(row + (4 * j + g) * E + e) =
            make_float4(f[j * E + e], f[j * E + e + 1], f[j * E + e + 2], f[j * E + e + 3]);
  }
};

// 0 where every value is finite, otherwise NaN
template <int N>
__device__ __forceinline__ float not_finite(const float* f, float t) {
#pragma unroll
  for (int i = 0; i < N; ++i) t = fmaf(f[i], 0.f, t);
  return t;
}

// acc += rows^T w over the chunk's 16 tokens, only those in the window: the path
// of a chunk with a value that is not finite.  row(j, r, e): channel e of token
// 4j + r of the chunk.
template <int CPL, typename F>
__device__ __forceinline__ void add_in_window(f32x4 (&acc)[CPL], const float* w, const bool* in, int m, int g, F row) {
#pragma unroll 1
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float wj = __shfl(w[r], 16 * j + m);
      const bool use = __shfl(in[r] ? 1 : 0, 16 * j + m) != 0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c][i] = use ? fmaf(wj, row(j, r, CPL * (4 * g + i) + c), acc[c][i]) : acc[c][i];
    }
}

template <int CPL>
__device__ __forceinline__ void add_product(f32x4 (&acc)[CPL], const float (&a)[4][CPL], const float* w) {
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < CPL; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r][c], w[r], acc[c], 0, 0, 0);
}

template <int N>
__device__ __forceinline__ f32x4 contract(const float* a, const float* b) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < N; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], s, 0, 0, 0);
  return s;
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Consecutive tiles stay on one XCD (blocks are handed to the eight XCDs in turn): they share most of their box.
__device__ __forceinline__ uint32_t xcd_block() {
  const uint32_t n = gridDim.x, q = n / 8, r = n % 8, x = blockIdx.x % 8;
  return x * q + min(x, r) + blockIdx.x / 8;
}

// The wave's tile; waves past the last tile repeat it and store nothing.
__device__ __forceinline__ uint32_t wave_tile(const AnyDims& d, int wave, int& part, bool& store) {
  const int per = 4 / d.split;
  const uint32_t t = xcd_block() * per + wave / d.split, n = (uint32_t)d.tiles;
  part = wave % d.split;
  store = t < n && part == 0;
  return min(t, n - 1);
}

// ---- forward ---------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(256) na3d_any_fwd_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                           const T* __restrict__ v, const float2* __restrict__ cs,
                                                           T* __restrict__ out, float* __restrict__ lse, AnyDims d,
                                                           const T* __restrict__ gate, int gate_dim) {
  using Fr = Frag<T, D>;
  constexpr int CPL = D / 16, NS = 4 * CPL + 2;
  __shared__ float merge[3 * 64 * NS];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  int part;
  bool store;
  const uint32_t tile = wave_tile(d, wave, part, store);
  const Walk w = Walk::make<false>(d, tile, m);
  const int64_t n_tok = (int64_t)d.Z * d.H * d.W, base = w.bh * n_tok;
  const uint32_t mine = w.mine();
  const float2* ph = cs ? cs + (int64_t)w.b * d.H * d.W * (D / 2) : nullptr;
  const T *kb = k + base * D, *vb = v + base * D;

  float qf[Fr::N];
  Fr::load(q + (base + mine) * D, g, qf);
  if (ph) Fr::rotate(ph + (int64_t)w.mine_in_plane() * (D / 2), g, qf);
  if (d.norm) Fr::normalise(qf, d.eps);
  const float qs = d.scale * kLog2e;
#pragma unroll
  for (int i = 0; i < Fr::N; ++i) qf[i] *= qs;

  f32x4 acc[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mx = kLowest, l = 0.f;
#pragma unroll 1
  for (uint32_t i0 = 16 * part; i0 < w.n; i0 += 16 * d.split) {
    int bz, by, bx;
    w.at(min(i0 + m, w.n - 1), bz, by, bx);
    const uint32_t p = w.plane(by, bx);
    float kf[Fr::N];
    Fr::load(kb + (int64_t)w.tok(bz, p) * D, g, kf);
    uint32_t tk[4];
    bool in[4];
    w.four(i0 + 4 * g, tk, in);
    float va[4][CPL];
#pragma unroll
    for (int r = 0; r < 4; ++r) load_n<T, CPL>(vb + (int64_t)tk[r] * D + m * CPL, va[r]);
    if (ph) Fr::rotate(ph + (int64_t)p * (D / 2), g, kf);
    if (d.norm) Fr::normalise(kf, d.eps);
    const f32x4 s = contract<Fr::N>(kf, qf);
    float sv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) sv[r] = in[r] ? s[r] : -INFINITY;
    // the reference moves only when a score exceeds it by more than 16: weights stay below 2^16
    const float top = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    if (__any(top > mx + 16.f)) {
      const float mn = fmaxf(mx, mfma::max_over_rows(top)), a = __builtin_amdgcn_exp2f(mx - mn);
      l *= a;
#pragma unroll
      for (int c = 0; c < CPL; ++c) acc[c] *= a;
      mx = mn;
    }
    float pw[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pw[r] = __builtin_amdgcn_exp2f(sv[r] - mx);
      l += pw[r];
    }
    float bad = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) bad = not_finite<CPL>(va[r], bad);
    if (__any(bad != 0.f)) {
      add_in_window<CPL>(acc, pw, in, m, g, [&](int j, int r, int e) {
        return ldf(vb + (int64_t)(uint32_t)__shfl((int)tk[r], 16 * j) * D + e);
      });
    } else {
      add_product<CPL>(acc, va, pw);
    }
  }
  l = sum_over_rows(l);
  if (d.split > 1) {  // merge the waves of a tile: common reference, then sums
    if (part > 0) {
      float* buf = merge + (wave - wave / d.split - 1) * (64 * NS) + lane;
#pragma unroll
      for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) buf[(4 * c + r) * 64] = acc[c][r];
      buf[(NS - 2) * 64] = mx;
      buf[(NS - 1) * 64] = l;
    }
    __syncthreads();
    if (part == 0) {
      for (int o = 1; o < d.split; ++o) {
        const float* from = merge + (wave - wave / d.split + o - 1) * (64 * NS) + lane;
        const float mo = from[(NS - 2) * 64], mn = fmaxf(mx, mo);
        const float a = __builtin_amdgcn_exp2f(mx - mn), b = __builtin_amdgcn_exp2f(mo - mn);
        l = l * a + from[(NS - 1) * 64] * b;
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[c][r] = acc[c][r] * a + from[(4 * c + r) * 64] * b;
        mx = mn;
      }
    }
  }
  if (!store || !w.live) return;
  const float inv = 1.f / l;
  float o[4 * CPL];
  const int64_t row = base + mine;
  const T* gp = gate ? gate + (gate_dim == 1 ? row : row * D + 4 * CPL * g) : nullptr;
  const float g1 = gate && gate_dim == 1 ? 1.f / (1.f + expf(-ldf(gp))) : 1.f;
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
      float x = acc[c][r] * inv;
      if (gate) x *= gate_dim == 1 ? g1 : 1.f / (1.f + expf(-ldf(gp + CPL * r + c)));
      o[CPL * r + c] = x;
    }
  store_n<T, 4 * CPL>(out + row * D + 4 * CPL * g, o);
  if (lse && g == 0) lse[row] = mx * kLn2 + logf(l);
}

// The lane's 4 CPL channels of a gradient row in the rotated, normalised frame,
// turned back (R^T, then the norm's Jacobian dx = r (dx^ - x^ mean(dx^ x^)),
// x^ = r x, x the raw row), and stored.
template <typename T, int D>
__device__ __forceinline__ void finish_row(const f32x4 (&acc)[D / 16], float mul, const T* raw, const float2* ph,
                                           const AnyDims& d, int g, bool store, T* dst) {
  constexpr int CPL = D / 16, N = 4 * CPL;
  float x[N];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < CPL; ++c) x[CPL * r + c] = acc[c][r] * mul;
  if (ph) {
#pragma unroll
    for (int t = 0; t < N; t += 4) {
      const float4 p = *reinterpret_cast<const float4*>(ph + (N * g + t) / 2);
      const float a = x[t], b = x[t + 1], c = x[t + 2], e = x[t + 3];
      x[t] = fmaf(a, p.x, b * p.y);
      x[t + 1] = fmaf(b, p.x, -a * p.y);
      x[t + 2] = fmaf(c, p.z, e * p.w);
      x[t + 3] = fmaf(e, p.z, -c * p.w);
    }
  }
  if (d.norm) {
    float u[N], ss = 0.f, dot = 0.f;
#pragma unroll
    for (int t = 0; t < N; t += Frag<T, D>::E) load_n<T, Frag<T, D>::E>(raw + N * g + t, u + t);
#pragma unroll
    for (int t = 0; t < N; ++t) ss = fmaf(u[t], u[t], ss);
    const float r = 1.f / sqrtf(sum_over_rows(ss) / D + d.eps);
#pragma unroll
    for (int t = 0; t < N; ++t) {
      u[t] *= r;
      dot = fmaf(x[t], u[t], dot);
    }
    dot = sum_over_rows(dot) / D;
#pragma unroll
    for (int t = 0; t < N; ++t) x[t] = r * fmaf(-u[t], dot, x[t]);
  }
  if (store) store_n<T, N>(dst + N * g, x);
}

// Sum of a tile's accumulators over the waves that share it, into the first of
// them; buf: 64 * 4 CPL floats per wave of the block.
template <int CPL>
__device__ __forceinline__ void merge_waves(f32x4 (&acc)[CPL], float* buf, int stride, int wave, int part, int split,
                                            int lane) {
  if (part > 0) {
#pragma unroll
    for (int c = 0; c < CPL; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) buf[wave * stride + (4 * c + r) * 64 + lane] = acc[c][r];
  }
  __syncthreads();
  if (part == 0)
    for (int o = 1; o < split; ++o)
#pragma unroll
      for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[c][r] += buf[(wave + o) * stride + (4 * c + r) * 64 + lane];
}

// ---- dq --------------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(256) na3d_any_dq_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                          const T* __restrict__ v, const float2* __restrict__ cs,
                                                          const T* __restrict__ dout, const T* __restrict__ dlo,
                                                          const float* __restrict__ lse, const float* __restrict__ dvec,
                                                          T* __restrict__ dq, AnyDims d) {
  using Fr = Frag<T, D>;
  constexpr int CPL = D / 16, LD = D + 4;
  __shared__ __attribute__((aligned(16))) float lds[4 * 16 * LD];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  int part;
  bool store;
  const uint32_t tile = wave_tile(d, wave, part, store);
  const Walk w = Walk::make<false>(d, tile, m);
  const int64_t n_tok = (int64_t)d.Z * d.H * d.W, base = w.bh * n_tok;
  const uint32_t mine = w.mine();
  const float2* ph = cs ? cs + (int64_t)w.b * d.H * d.W * (D / 2) : nullptr;
  const float2* phq = ph ? ph + (int64_t)w.mine_in_plane() * (D / 2) : nullptr;
  const T *kb = k + base * D, *vb = v + base * D;
  const int64_t row = base + mine;
  float* kt = lds + wave * 16 * LD;

  float qf[Fr::N], gf[Fr::N];
  Fr::load(q + row * D, g, qf);
  if (phq) Fr::rotate(phq, g, qf);
  if (d.norm) Fr::normalise(qf, d.eps);
  const float qs = d.scale * kLog2e;
#pragma unroll
  for (int i = 0; i < Fr::N; ++i) qf[i] *= qs;
  Fr::load(dout + row * D, g, gf);
  if (dlo) {
    float lf[Fr::N];
    Fr::load(dlo + row * D, g, lf);
#pragma unroll
    for (int i = 0; i < Fr::N; ++i) gf[i] += lf[i];
  }
  const float L = lse[row], Dv = dvec[row];
  f32x4 acc[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (uint32_t i0 = 16 * part; i0 < w.n; i0 += 16 * d.split) {
    int bz, by, bx;
    w.at(min(i0 + m, w.n - 1), bz, by, bx);
    const uint32_t p = w.plane(by, bx), t = w.tok(bz, p);
    float kf[Fr::N], vf[Fr::N];
    Fr::load(kb + (int64_t)t * D, g, kf);
    Fr::load(vb + (int64_t)t * D, g, vf);
    uint32_t tk[4];
    bool in[4];
    w.four(i0 + 4 * g, tk, in);
    if (ph) Fr::rotate(ph + (int64_t)p * (D / 2), g, kf);
    if (d.norm) Fr::normalise(kf, d.eps);
    wave_lds_fence();  // the last chunk's reads are done
    Fr::to_lds(kt + m * LD, g, kf);
    const f32x4 s = contract<Fr::N>(kf, qf);
    const f32x4 y = contract<Fr::N>(vf, gf);
    float ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float pw = __builtin_amdgcn_exp2f(fmaf(-L, kLog2e, s[r]));
      ds[r] = in[r] ? pw * (y[r] - Dv) : 0.f;
    }
    wave_lds_fence();
    if (__any(not_finite<Fr::N>(kf, 0.f) != 0.f)) {
      add_in_window<CPL>(acc, ds, in, m, g, [&](int j, int r, int e) { return kt[(4 * j + r) * LD + e]; });
    } else {
      float ka[4][CPL];
#pragma unroll
      for (int r = 0; r < 4; ++r) load_n<float, CPL>(kt + (4 * g + r) * LD + m * CPL, ka[r]);
      add_product<CPL>(acc, ka, ds);
    }
  }
  if (d.split > 1) {
    __syncthreads();
    merge_waves<CPL>(acc, lds, 16 * LD, wave, part, d.split, lane);
  }
  if (store) finish_row<T, D>(acc, d.scale, q + row * D, phq, d, g, w.live, dq + row * D);
}

// ---- dk, dv ----------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(256) na3d_any_dkdv_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                            const T* __restrict__ v, const float2* __restrict__ cs,
                                                            const T* __restrict__ dout, const T* __restrict__ dlo,
                                                            const float* __restrict__ lse, const float* __restrict__ dvec,
                                                            T* __restrict__ dk, T* __restrict__ dv, AnyDims d) {
  using Fr = Frag<T, D>;
  constexpr int CPL = D / 16, LD = D + 4, WAVE = 2 * 16 * LD + 32;
  __shared__ __attribute__((aligned(16))) float lds[4 * WAVE];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  int part;
  bool store;
  const uint32_t tile = wave_tile(d, wave, part, store);
  const Walk w = Walk::make<true>(d, tile, m);
  const int64_t n_tok = (int64_t)d.Z * d.H * d.W, base = w.bh * n_tok;
  const uint32_t mine = w.mine();
  const float2* ph = cs ? cs + (int64_t)w.b * d.H * d.W * (D / 2) : nullptr;
  const float2* phk = ph ? ph + (int64_t)w.mine_in_plane() * (D / 2) : nullptr;
  const T *qb = q + base * D, *gb = dout + base * D, *lb = dlo ? dlo + base * D : nullptr;
  const int64_t row = base + mine;
  float *qt = lds + wave * WAVE, *gt = qt + 16 * LD, *st = gt + 16 * LD;

  float kf[Fr::N], vf[Fr::N];
  Fr::load(k + row * D, g, kf);
  if (phk) Fr::rotate(phk, g, kf);
  if (d.norm) Fr::normalise(kf, d.eps);
  Fr::load(v + row * D, g, vf);
  const float qs = d.scale * kLog2e;
  f32x4 ak[CPL], av[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) ak[c] = av[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
  for (uint32_t i0 = 16 * part; i0 < w.n; i0 += 16 * d.split) {
    int bz, by, bx;
    w.at(min(i0 + m, w.n - 1), bz, by, bx);
    const uint32_t p = w.plane(by, bx), t = w.tok(bz, p);
    float qf[Fr::N], gf[Fr::N];
    Fr::load(qb + (int64_t)t * D, g, qf);
    Fr::load(gb + (int64_t)t * D, g, gf);
    const float stat = g == 0 ? lse[base + t] : g == 1 ? dvec[base + t] : 0.f;
    if (lb) {
      float lf[Fr::N];
      Fr::load(lb + (int64_t)t * D, g, lf);
#pragma unroll
      for (int i = 0; i < Fr::N; ++i) gf[i] += lf[i];
    }
    uint32_t tk[4];
    bool in[4];
    w.four(i0 + 4 * g, tk, in);
    if (ph) Fr::rotate(ph + (int64_t)p * (D / 2), g, qf);
    if (d.norm) Fr::normalise(qf, d.eps);
#pragma unroll
    for (int i = 0; i < Fr::N; ++i) qf[i] *= qs;
    wave_lds_fence();  // the last chunk's reads are done
    Fr::to_lds(qt + m * LD, g, qf);
    Fr::to_lds(gt + m * LD, g, gf);
    if (g < 2) st[lane] = stat;
    const f32x4 s = contract<Fr::N>(qf, kf);
    const f32x4 y = contract<Fr::N>(gf, vf);
    wave_lds_fence();
    const float4 L = *reinterpret_cast<const float4*>(st + 4 * g), Dv = *reinterpret_cast<const float4*>(st + 16 + 4 * g);
    const float Ls[4] = {L.x, L.y, L.z, L.w}, Ds[4] = {Dv.x, Dv.y, Dv.z, Dv.w};
    float pw[4], ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pw[r] = in[r] ? __builtin_amdgcn_exp2f(fmaf(-Ls[r], kLog2e, s[r])) : 0.f;
      ds[r] = in[r] ? pw[r] * (y[r] - Ds[r]) : 0.f;
    }
    if (__any(not_finite<Fr::N>(qf, not_finite<Fr::N>(gf, 0.f)) != 0.f)) {
      add_in_window<CPL>(av, pw, in, m, g, [&](int j, int r, int e) { return gt[(4 * j + r) * LD + e]; });
      add_in_window<CPL>(ak, ds, in, m, g, [&](int j, int r, int e) { return qt[(4 * j + r) * LD + e]; });
    } else {
      float a[4][CPL];
#pragma unroll
      for (int r = 0; r < 4; ++r) load_n<float, CPL>(gt + (4 * g + r) * LD + m * CPL, a[r]);
      add_product<CPL>(av, a, pw);
#pragma unroll
      for (int r = 0; r < 4; ++r) load_n<float, CPL>(qt + (4 * g + r) * LD + m * CPL, a[r]);
      add_product<CPL>(ak, a, ds);
    }
  }
  if (d.split > 1) {
    __syncthreads();
    merge_waves<CPL>(ak, lds, WAVE, wave, part, d.split, lane);
    merge_waves<CPL>(av, lds + 16 * LD, WAVE, wave, part, d.split, lane);
  }
  if (!store) return;
  // the staged queries carry scale log2(e)
  finish_row<T, D>(ak, kLn2, k + row * D, phk, d, g, w.live, dk + row * D);
  if (w.live) {
    float o[4 * CPL];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < CPL; ++c) o[CPL * r + c] = av[c][r];
    store_n<T, 4 * CPL>(dv + row * D + 4 * CPL * g, o);
  }
}

// D_i = <dout_i, out_i> in float32.  A lane reads one 16-byte piece of a row of
// both tensors; the CPR lanes of a row (aligned within the wave) add their
// partial sums by butterfly exchanges.
template <typename T, int D>
__global__ void __launch_bounds__(256) na3d_bwd_pre_kernel(const T* __restrict__ out, const T* __restrict__ dout,
                                                           float* __restrict__ dvec, int64_t nq) {
  constexpr int E = 16 / (int)sizeof(T);  // elements per 16-byte piece
  constexpr int CPR = D / E;              // pieces per row: 4, 8 or 16
  static_assert(64 % CPR == 0, "a row's lanes must not straddle a wave");
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = gid / CPR;
  const int c = (int)(gid % CPR);
  float acc = 0.f;
  if (row < nq) {
    float a[E], b[E];
    load_n<T, E>(out + row * D + c * E, a);
    load_n<T, E>(dout + row * D + c * E, b);
#pragma unroll
    for (int e = 0; e < E; ++e) acc = fmaf(b[e], a[e], acc);
  }
#pragma unroll
  for (int off = CPR / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if (row < nq && c == 0) dvec[row] = acc;
}

dim3 any_grid(const AnyDims& a) {
  const int per = 4 / a.split;
  return dim3((uint32_t)((a.tiles + per - 1) / per));
}

template <typename T, int D>
void fwd_any(const strata_na3d_desc& d, const NaOpts& o, const void* q, const void* k, const void* v, const float* cs,
             void* out, float* lse, hipStream_t s) {
  const AnyDims a = any_dims(d.B, d.heads, d.Z, d.H, d.W, d.kz, d.ky, d.kx, d.scale, o.qk_norm, o.eps);
  hipLaunchKernelGGL((na3d_any_fwd_kernel<T, D>), any_grid(a), dim3(256), 0, s, static_cast<const T*>(q),
                     static_cast<const T*>(k), static_cast<const T*>(v), reinterpret_cast<const float2*>(cs),
                     static_cast<T*>(out), lse, a, static_cast<const T*>(o.gate), o.gate_dim);
}

template <typename T, int D>
void bwd_any(int part, const strata_na3d_desc& d, const BwdOpts& o, const void* q, const void* k, const void* v,
             const float* cs, const void* out, const void* dout, const float* lse, void* dq, void* dk, void* dv,
             float* dvec, hipStream_t s) {
  const float2* c2 = reinterpret_cast<const float2*>(cs);
  if (part == 0) {
    const int64_t n = (int64_t)d.B * d.heads * d.Z * d.H * d.W;
    hipLaunchKernelGGL((na3d_bwd_pre_kernel<T, D>), dim3((int)((n * (D * sizeof(T) / 16) + 255) / 256)), dim3(256), 0,
                       s, static_cast<const T*>(out), static_cast<const T*>(dout), dvec, n);
    return;
  }
  const AnyDims a = any_dims(d.B, d.heads, d.Z, d.H, d.W, d.kz, d.ky, d.kx, d.scale, o.qk_norm, o.eps);
  if (part == 1)
    hipLaunchKernelGGL((na3d_any_dq_kernel<T, D>), any_grid(a), dim3(256), 0, s, static_cast<const T*>(q),
                       static_cast<const T*>(k), static_cast<const T*>(v), c2, static_cast<const T*>(dout),
                       static_cast<const T*>(o.dout_lo), lse, dvec, static_cast<T*>(dq), a);
  else
    hipLaunchKernelGGL((na3d_any_dkdv_kernel<T, D>), any_grid(a), dim3(256), 0, s, static_cast<const T*>(q),
                       static_cast<const T*>(k), static_cast<const T*>(v), c2, static_cast<const T*>(dout),
                       static_cast<const T*>(o.dout_lo), lse, dvec, static_cast<T*>(dk), static_cast<T*>(dv), a);
}

}  // namespace

bool na3d_any_takes(const strata_na3d_desc& d) {
  return any_fits(d.B, d.heads, d.Z, d.H, d.W, d.kz, d.ky, d.kx);
}

void launch_na3d_fwd_any(const strata_na3d_desc& d, const NaOpts& o, const void* q, const void* k, const void* v,
                         const float* cs, void* out, float* lse, hipStream_t s) {
  if (d.dtype == STRATA_BF16) {
    if (d.head_dim == 32) fwd_any<uint16_t, 32>(d, o, q, k, v, cs, out, lse, s);
    else if (d.head_dim == 64) fwd_any<uint16_t, 64>(d, o, q, k, v, cs, out, lse, s);
    else fwd_any<uint16_t, 128>(d, o, q, k, v, cs, out, lse, s);
  } else {
    if (d.head_dim == 32) fwd_any<float, 32>(d, o, q, k, v, cs, out, lse, s);
    else if (d.head_dim == 64) fwd_any<float, 64>(d, o, q, k, v, cs, out, lse, s);
    else fwd_any<float, 128>(d, o, q, k, v, cs, out, lse, s);
  }
}

void launch_na3d_bwd_any(int part, const strata_na3d_desc& d, const BwdOpts& o, const void* q, const void* k,
                         const void* v, const float* cs, const void* out, const void* dout, const float* lse, void* dq,
                         void* dk, void* dv, float* dvec, hipStream_t s) {
  if (d.dtype == STRATA_BF16) {
    if (d.head_dim == 32) bwd_any<uint16_t, 32>(part, d, o, q, k, v, cs, out, dout, lse, dq, dk, dv, dvec, s);
    else if (d.head_dim == 64) bwd_any<uint16_t, 64>(part, d, o, q, k, v, cs, out, dout, lse, dq, dk, dv, dvec, s);
    else bwd_any<uint16_t, 128>(part, d, o, q, k, v, cs, out, dout, lse, dq, dk, dv, dvec, s);
  } else {
    if (d.head_dim == 32) bwd_any<float, 32>(part, d, o, q, k, v, cs, out, dout, lse, dq, dk, dv, dvec, s);
    else if (d.head_dim == 64) bwd_any<float, 64>(part, d, o, q, k, v, cs, out, dout, lse, dq, dk, dv, dvec, s);
    else bwd_any<float, 128>(part, d, o, q, k, v, cs, out, dout, lse, dq, dk, dv, dvec, s);
  }
}

}  // namespace strata
