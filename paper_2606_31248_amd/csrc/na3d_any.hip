// Neighbourhood attention for every problem without a 16-bit MFMA kernel: both
// dtypes, head_dim 32, 64 or 128, any window and grid.  All arithmetic is
// float32; the contractions run on the float32 matrix instruction
// v_mfma_f32_16x16x4_f32 (2048 FLOP per instruction, 154 TFLOP/s measured with
// a large matrix product), so nothing is rounded to 16 bits between the inputs
// and the results.
//
// A workgroup owns a tile of 16 tokens (queries in the forward and dq, keys in
// dk/dv), a block of (z, y, x) extents whose product is 16; its four waves take
// the tile in four (batch, head) grids, or share its work in two or one.  A wave
// walks the box of tokens on the other side that any of the 16 sees, 16 at a time
// (a chunk), in linear order over the whole three-dimensional box, so that at most
// one chunk is padded; positions and window masks, the same in every grid, are
// formed once by the four waves in LDS.  What bounds it: matrix and vector
// instructions add up (a float32 matrix instruction takes 32 cycles, head_dim / 4
// of them per chunk and product), times the share of the box outside the windows.
//
// Layouts (lane l, m = l % 16, g = l / 16).  A 16 x 4 operand gives lane l row m,
// column g.  The sum over head_dim may take the channels in any order, so lane l
// holds the 16-byte pieces g, g + 4, ... of row m (whole pieces, one load each)
// and step s of the contraction takes element s of both operands.  The scores
// come out with the tile's token as the column m and the chunk's tokens 4g + r as
// the rows, which is the operand layout of the second product as it stands; its
// other operand holds, for token 4g + r, the head_dim / 16 channels from
// m head_dim / 16 on, so that output tile c, row m is channel m head_dim / 16 + c.
// A chunk's rows are loaded with four neighbouring lanes to a row (64 bytes
// together; in the operand layout neighbouring lanes hold different rows, every
// lane its own access, and the vector cache's access rate bounded the kernels),
// rotated and normalised there, and pass through the wave's own part of LDS into
// the operand layout, in the backward also into the other one.
//
// Measured against one thread per query (or one wave per query below 2^18) with
// float32 vector arithmetic: float32 forward and backward, 4 heads x 7x21x27,
// d 64, 5x9x9: 14733 -> 217 us; bf16 3x3x3 forward and backward, 6 tiles x 16
// heads x 24x16x16: 20589 -> 763 us (about 350 us more with each wave forming its
// own positions and masks, 260 with every product in float32, 115 with rows
// loaded in the operand layout); float32 forward,
// 4 heads x 4x16x16, d 32, 3x7x7: 56.8 -> 9.0 us.
//
// Scores stay in natural units and are taken less the running maximum or the lse
// before the exponential, so that a weight's error does not grow with its score; the
// error of out and the gradients against 64 bits is below that of the scalar kernels,
// that of lse its own rounding (0 to 3% of the times above go into this).
//
// Waves per SIMD asked for (launch bounds): at head_dim 64 with bf16 rows four (the
// forward, dQ) and three, which two registers in scratch buy: the 3x3x3 case takes
// 824 us without the bounds.  For float32 rows the bounds of head_dim 64 are what the
// compiler takes by itself; at head_dim 32 there are four and more without one; at
// head_dim 128 none is asked for (one or two waves).
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

constexpr float kLowest = -3.402823466e38f;

// e^x for x <= 0 (but for rounding), within 2 ulp: x log2(e) in two terms, 2^hi
// (1 + lo ln 2), as the rounding of the product alone would show in every weight.
// 0 below -104 (and at -inf, whose terms have no sum); NaN stays.
__device__ __forceinline__ float exp_of(float x) {
  constexpr float kHi = 1.44269504f, kLo = 1.925963033e-8f, kLn2 = 0.6931471805599453f;  // log2(e) = kHi + kLo
  const float h = x * kHi, lo = fmaf(x, kLo, fmaf(x, kHi, -h)), e = __builtin_amdgcn_exp2f(h);
  return x < -104.f ? 0.f : fmaf(e, lo * kLn2, e);
}

template <typename T>
__device__ __forceinline__ float ldf(const T* p);
template <>
__device__ __forceinline__ float ldf<float>(const float* p) { return *p; }
template <>
__device__ __forceinline__ float ldf<uint16_t>(const uint16_t* p) { return bf16_to_f32(*p); }

// N values from their storage words
template <typename T, int N>
__device__ __forceinline__ void widen_n(const uint32_t* u, float* f) {
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
  widen_n<T, N>(u, f);
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

// Sum over each aligned group of four lanes
__device__ __forceinline__ float sum_over_quad(float x) {
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, false));  // quad_perm 1,0,3,2
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, false));  // quad_perm 2,3,0,1
  return x;
}

// The lane's share of a row in the operand layout: pieces g, g + 4, ... of 16 bytes
template <typename T, int D>
struct Frag {
  static constexpr int E = 16 / (int)sizeof(T);  // elements of a piece
  static constexpr int NP = D / (4 * E);         // pieces per lane
  static constexpr int N = D / 4;                // elements per lane
  struct Raw {
    uint4 v[NP];
  };
  struct Phases {
    float4 v[N / 4];
  };
  static __device__ __forceinline__ void load(const T* row, int g, Raw& r) {
#pragma unroll
    for (int j = 0; j < NP; ++j) r.v[j] = *reinterpret_cast<const uint4*>(row + (4 * j + g) * E);
  }
  static __device__ __forceinline__ void widen(const Raw& r, float* f) {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      const uint32_t u[4] = {r.v[j].x, r.v[j].y, r.v[j].z, r.v[j].w};
      widen_n<T, E>(u, f + j * E);
    }
  }
  static __device__ __forceinline__ void load(const T* row, int g, float* f) {
    Raw r;
    load(row, g, r);
    widen(r, f);
  }
  static __device__ __forceinline__ void load_phases(const float2* ph, int g, Phases& p) {
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int e = 0; e < E; e += 4)
        p.v[(j * E + e) / 4] = *reinterpret_cast<const float4*>(ph + ((4 * j + g) * E + e) / 2);
  }
  static __device__ __forceinline__ void rotate(const float2* ph, int g, float* f) {
    Phases p;
    load_phases(ph, g, p);
    rotate(p, f);
  }
  static __device__ __forceinline__ void rotate(const Phases& ph, float* f) {
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int e = 0; e < E; e += 4) {
        const float4 p = ph.v[(j * E + e) / 4];
        float* x = f + j * E + e;
        const float a = x[0], b = x[1], c = x[2], d = x[3];
        x[0] = fmaf(a, p.x, -b * p.y);
        x[1] = fmaf(a, p.y, b * p.x);
        x[2] = fmaf(c, p.z, -d * p.w);
        x[3] = fmaf(c, p.w, d * p.z);
      }
  }
  // QK RMSNorm: divide the row by its root mean square, its four lanes together
  // (QUAD: they are neighbours, the loading layout; else 16 lanes apart)
  template <bool QUAD>
  static __device__ __forceinline__ void normalise(float* f, float eps) {
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) ss = fmaf(f[i], f[i], ss);
    const float x = (QUAD ? sum_over_quad(ss) : sum_over_rows(ss)) * (1.f / D) + eps;
    // within an ulp like the division by the root, which takes the ends of the
    // range (and 20 more instructions)
    float r = __builtin_amdgcn_rsqf(x);
    if (__any(!(x > 1e-30f && x < 1e30f))) r = 1.f / sqrtf(x);
#pragma unroll
    for (int i = 0; i < N; ++i) f[i] *= r;
  }
  static __device__ __forceinline__ void from_lds(const float* row, int g, float* f) {
#pragma unroll
    for (int j = 0; j < NP; ++j) load_n<float, E>(row + (4 * j + g) * E, f + j * E);
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

// Channel of element i of a lane's output tile c: the lane holds the 4 CPL
// channels from 4 CPL g on, tile by tile with products of bf16 rows (X), element
// by element with float32 ones.
template <int CPL, bool X>
__device__ __forceinline__ constexpr int channel(int g, int c, int i) {
  return 4 * CPL * g + (X ? 4 * c + i : CPL * i + c);
}

// ---- products with rows that are bf16 as they come ----------------------------
// A product of two bf16 values is exact in float32, so V . dO^T takes the raw
// rows on the bf16 instruction (16 times the float32 rate), and P . V, dO^T . P
// take the float32 weights as three bf16 terms that add up to them (8 bits each,
// 2^-25 left) against the raw rows: sums of exact products in float32, as before.
template <int NP>
__device__ __forceinline__ f32x4 contract16(const uint4 (&a)[NP], const uint4 (&b)[NP]) {
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < NP; ++j)
    s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(mfma::bf16x8, a[j]),
                                                __builtin_bit_cast(mfma::bf16x8, b[j]), s, 0, 0, 0);
  return s;
}

// bytes of a staged bf16 row
constexpr int row16(int D) { return 2 * D + 16; }

// the lane's pieces of row m of a chunk, to and from its wave's tile of bf16 rows
template <int NP>
__device__ __forceinline__ void to_lds16(char* tile, int m, int g, const uint4 (&r)[NP]) {
#pragma unroll
  for (int j = 0; j < NP; ++j) mfma::st16(tile + m * row16(32 * NP) + 16 * (4 * j + g), r[j]);
}
template <int NP>
__device__ __forceinline__ void from_lds16(const char* tile, int m, int g, uint4 (&r)[NP]) {
#pragma unroll
  for (int j = 0; j < NP; ++j) r[j] = mfma::ld16(tile + m * row16(32 * NP) + 16 * (4 * j + g));
}

// acc += rows^T w, rows: the wave's tile of bf16 rows, read transposed (tile c,
// row m: channel 4 CPL (m / 4) + 4 c + m % 4)
template <int CPL>
__device__ __forceinline__ void add_product16(f32x4 (&acc)[CPL], const char* tile, int m, int g, const float* w) {
  mfma::i16x4 t[3];
  float x[4] = {w[0], w[1], w[2], w[3]};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const uint32_t a = mfma::pack2(x[0], x[1]), b = mfma::pack2(x[2], x[3]);
    t[k] = __builtin_bit_cast(mfma::i16x4, make_uint2(a, b));
    x[0] -= mfma::lo_bf16(a);
    x[1] -= mfma::hi_bf16(a);
    x[2] -= mfma::lo_bf16(b);
    x[3] -= mfma::hi_bf16(b);
  }
  const char* p = tile + (4 * g + (m >> 2)) * row16(16 * CPL) + 8 * CPL * (m & 3);
#pragma unroll
  for (int c = 0; c < CPL; ++c) {
    const mfma::i16x4 r = mfma::tr_read(p + 8 * c);
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(r, t[k], acc[c], 0, 0, 0);
  }
}

// acc += rows^T w over the chunk's 16 tokens, only those in the window: the path
// of a chunk with a value that is not finite.  row(j, r, e): channel e of token
// 4j + r of the chunk.
template <int CPL, bool X, typename F>
__device__ __forceinline__ void add_in_window(f32x4 (&acc)[CPL], const float* w, uint32_t see, int m, int g, F row) {
#pragma unroll 1
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float wj = __shfl(w[r], 16 * j + m);
      const bool use = (__shfl((int)see, 16 * j + m) >> r) & 1;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c][i] = use ? fmaf(wj, row(j, r, channel<CPL, X>(g, c, i)), acc[c][i]) : acc[c][i];
    }
}

// acc += rows^T w with float32 rows.  TWO (the float32 forward): the chunk is summed
// by itself first, so that the sums over a box round in two levels (error of the
// output at 9x9x9, d 32: 3.1e-7 in one level, 2.1e-7 in two, 2.4e-7 with 64 lanes
// per query; the gradients' is below that of one thread per query with one level).
template <bool TWO, int CPL>
__device__ __forceinline__ void add_product(f32x4 (&acc)[CPL], const float (&a)[4][CPL], const float* w) {
  f32x4 t[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) t[c] = TWO ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[c];
#pragma unroll
  for (int r = 0; r < 4; ++r)
#pragma unroll
    for (int c = 0; c < CPL; ++c) t[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r][c], w[r], t[c], 0, 0, 0);
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = TWO ? acc[c] + t[c] : t[c];
}

// two sums of every other step: half as many roundings in a row as one
template <int N>
__device__ __forceinline__ f32x4 contract(const float* a, const float* b) {
  f32x4 s[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
  for (int i = 0; i < N; ++i) s[i & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], s[i & 1], 0, 0, 0);
  return s[0] + s[1];
}

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The workgroup's tile (a place in the grid), and the wave's grid (batch * heads +
// head) and part of the chunks; waves past the last grid repeat it and store nothing.
struct Place {
  uint32_t tile;
  int64_t bh;
  int b, part;
  bool store;
};
__device__ __forceinline__ Place wave_place(const AnyDims& d, uint32_t launched, int wave) {
  const uint32_t blk = xcd_order(launched, d.blocks), grp = d.places.div(blk), bh = grp * (4 / d.split) + wave / d.split;
  const uint32_t in = min(bh, d.nbh - 1);
  const int part = wave % d.split;
  return Place{blk - grp * d.places.n, (int64_t)in, (int)(in / (uint32_t)d.heads), part, bh < d.nbh && part == 0};
}

// body(c, see): every chunk of the wave's part of the box, in runs that the
// workgroup's waves fill together; c: the chunk's place in the run, see: the
// lane's four bits.  Every wave of the workgroup passes every barrier.
template <typename F>
__device__ __forceinline__ void walk_box(const Walk& w, Run& run, const AnyDims& d, int part, int lane, F body) {
#pragma unroll 1
  for (uint32_t i0 = 0; i0 < w.n; i0 += 16 * kRun) {
    if (i0) __syncthreads();
    fill_run(w, run, i0, threadIdx.x);
    __syncthreads();
    const uint32_t end = min((uint32_t)kRun, (w.n - i0 + 15) / 16);
#pragma unroll 1
    for (uint32_t c = part; c < end; c += d.split) body(c, run.see[64 * c + lane]);
  }
}

// x where bit r is set, else `other`
__device__ __forceinline__ float pick(uint32_t see, int r, float x, float other) {
  const uint32_t sel = (uint32_t)__builtin_amdgcn_sbfe((int)see, r, 1);
  return __uint_as_float((sel & __float_as_uint(x)) | (~sel & __float_as_uint(other)));
}

// ---- forward ---------------------------------------------------------------
template <typename T, int D>
__global__ void __launch_bounds__(256, D == 64 && sizeof(T) == 2 ? 4 : 1) na3d_any_fwd_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                           const T* __restrict__ v, const float2* __restrict__ cs,
                                                           T* __restrict__ out, float* __restrict__ lse, AnyDims d,
                                                           const T* __restrict__ gate, int gate_dim) {
  using Fr = Frag<T, D>;
  constexpr bool X = sizeof(T) == 2;
  constexpr int CPL = D / 16, NS = 4 * CPL + 2;
  constexpr int LD = D + 4, KB = 16 * LD * 4, WAVE = KB + (X ? 16 * row16(D) : 0);  // K~ rows, bf16 V rows
  static_assert(4 * WAVE >= 3 * 64 * NS * 4, "the merge of the waves fits the tiles");
  __shared__ __attribute__((aligned(16))) char tiles[4 * WAVE];
  float* const merge = reinterpret_cast<float*>(tiles);
  __shared__ __attribute__((aligned(16))) Run run;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const int lm = lane >> 2, lg = lane & 3;  // row and piece that the lane loads
  const uint32_t launched = blockIdx.y * gridDim.x + blockIdx.x;
  if (launched >= d.blocks) return;
  const Place at = wave_place(d, launched, wave);
  const int part = at.part;
  const Walk w = Walk::make<false>(d, at.tile, m);
  const int64_t n_tok = (int64_t)d.Z * d.H * d.W, base = at.bh * n_tok;
  const uint32_t mine = w.mine();
  const float2* ph = cs ? cs + (int64_t)at.b * d.H * d.W * (D / 2) : nullptr;
  const T *kb = k + base * D, *vb = v + base * D;

  float qf[Fr::N];
  Fr::load(q + (base + mine) * D, g, qf);
  if (ph) Fr::rotate(ph + (int64_t)w.mine_in_plane() * (D / 2), g, qf);
  if (d.norm) Fr::template normalise<false>(qf, d.eps);

  f32x4 acc[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mx = kLowest, l = 0.f;
  walk_box(w, run, d, part, lane, [&](uint32_t ch, uint32_t see) __attribute__((always_inline)) {
    float* const kt = reinterpret_cast<float*>(tiles + wave * WAVE);
    char* const tv = tiles + wave * WAVE + KB;
    float kf[Fr::N];
    Fr::load(kb + (int64_t)run.tok[16 * ch + lm] * D, lg, kf);
    float va[4][CPL];
    typename Fr::Raw vr;
    if constexpr (X) {
      Fr::load(vb + (int64_t)run.tok[16 * ch + lm] * D, lg, vr);
    } else {
      const uint4 t4 = *reinterpret_cast<const uint4*>(&run.tok[16 * ch + 4 * g]);
      const uint32_t tk[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
      for (int r = 0; r < 4; ++r) load_n<T, CPL>(vb + (int64_t)tk[r] * D + m * CPL, va[r]);
    }
    if (ph) Fr::rotate(ph + (int64_t)run.pl[16 * ch + lm] * (D / 2), lg, kf);
    if (d.norm) Fr::template normalise<true>(kf, d.eps);
    wave_lds_fence();  // the last chunk's reads are done
    Fr::to_lds(kt + lm * LD, lg, kf);
    if constexpr (X) to_lds16(tv, lm, lg, vr.v);
    wave_lds_fence();
    Fr::from_lds(kt + m * LD, g, kf);
    const f32x4 s = contract<Fr::N>(kf, qf);
    float sv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) sv[r] = pick(see, r, s[r] * d.scale, -INFINITY);
    // the reference is the largest score so far, as the weights' error grows with their distance from it
    const float top = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    if (__any(top > mx)) {
      const float mn = fmaxf(mx, mfma::max_over_rows(top)), a = exp_of(mx - mn);
      l *= a;
#pragma unroll
      for (int c = 0; c < CPL; ++c) acc[c] *= a;
      mx = mn;
    }
    float pw[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) pw[r] = exp_of(sv[r] - mx);
    l += (pw[0] + pw[1]) + (pw[2] + pw[3]);
    // not finite: a value of V (a product of its row with zeros shows it)
    float bad = 0.f;
    if constexpr (X) {  // (whichever lanes hold it)
      typename Fr::Raw zero;
#pragma unroll
      for (int j = 0; j < Fr::NP; ++j) zero.v[j] = make_uint4(0u, 0u, 0u, 0u);
      const f32x4 z = contract16(vr.v, zero.v);
      bad = z[0] + z[1] + z[2] + z[3];
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) bad = not_finite<CPL>(va[r], bad);
    }
    if (__any(bad != 0.f)) {
      add_in_window<CPL, X>(acc, pw, see, m, g, [&](int j, int r, int e) {
        return ldf(vb + (int64_t)run.tok[16 * ch + 4 * j + r] * D + e);
      });
    } else if constexpr (X) {
      add_product16<CPL>(acc, tv, m, g, pw);
    } else {
      add_product<true>(acc, va, pw);
    }
  });
  l = sum_over_rows(l);
  if (d.split > 1) {  // merge the waves of a tile: common reference, then sums
    __syncthreads();  // every tile has been read
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
        const float a = exp_of(mx - mn), b = exp_of(mo - mn);
        l = l * a + from[(NS - 1) * 64] * b;
#pragma unroll
        for (int c = 0; c < CPL; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[c][r] = acc[c][r] * a + from[(4 * c + r) * 64] * b;
        mx = mn;
      }
    }
  }
  if (!at.store || !w.live) return;
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
      const int e = channel<CPL, X>(0, c, r);
      if (gate) x *= gate_dim == 1 ? g1 : 1.f / (1.f + expf(-ldf(gp + e)));
      o[e] = x;
    }
  store_n<T, 4 * CPL>(out + row * D + 4 * CPL * g, o);
  if (lse && g == 0) lse[row] = mx + logf(l);
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
// X: bf16 rows and dO in one term
template <typename T, int D, bool X>
__global__ void __launch_bounds__(256, D == 64 ? (X ? 4 : 3) : 1) na3d_any_dq_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                          const T* __restrict__ v, const float2* __restrict__ cs,
                                                          const T* __restrict__ dout, const T* __restrict__ dlo,
                                                          const float* __restrict__ lse, const float* __restrict__ dvec,
                                                          T* __restrict__ dq, AnyDims d) {
  using Fr = Frag<T, D>;
  constexpr int CPL = D / 16, LD = D + 4, VT = X ? 4 * row16(D) : 16 * LD;  // floats of the V tile
  constexpr int WAVE = 16 * LD + VT;
  __shared__ __attribute__((aligned(16))) float lds[4 * WAVE];
  __shared__ __attribute__((aligned(16))) Run run;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const int lm = lane >> 2, lg = lane & 3;  // row and piece that the lane loads
  const uint32_t launched = blockIdx.y * gridDim.x + blockIdx.x;
  if (launched >= d.blocks) return;
  const Place at = wave_place(d, launched, wave);
  const int part = at.part;
  const Walk w = Walk::make<false>(d, at.tile, m);
  const int64_t n_tok = (int64_t)d.Z * d.H * d.W, base = at.bh * n_tok;
  const uint32_t mine = w.mine();
  const float2* ph = cs ? cs + (int64_t)at.b * d.H * d.W * (D / 2) : nullptr;
  const float2* phq = ph ? ph + (int64_t)w.mine_in_plane() * (D / 2) : nullptr;
  const T *kb = k + base * D, *vb = v + base * D;
  const int64_t row = base + mine;
  float *kt = lds + wave * WAVE, *vt = kt + 16 * LD;

  float qf[Fr::N], gf[Fr::N];
  Fr::load(q + row * D, g, qf);
  if (phq) Fr::rotate(phq, g, qf);
  if (d.norm) Fr::template normalise<false>(qf, d.eps);
  typename Fr::Raw gr;
  if constexpr (X) {
    Fr::load(dout + row * D, g, gr);
  } else {
    Fr::load(dout + row * D, g, gf);
    if (dlo) {
      float lf[Fr::N];
      Fr::load(dlo + row * D, g, lf);
#pragma unroll
      for (int i = 0; i < Fr::N; ++i) gf[i] += lf[i];
    }
  }
  const float L = lse[row], Dv = dvec[row];
  f32x4 acc[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  walk_box(w, run, d, part, lane, [&](uint32_t ch, uint32_t see) __attribute__((always_inline)) {
    const uint32_t t = run.tok[16 * ch + lm];
    float kf[Fr::N], vf[Fr::N];
    typename Fr::Raw vr;
    Fr::load(kb + (int64_t)t * D, lg, kf);
    if constexpr (X) Fr::load(vb + (int64_t)t * D, lg, vr);
    else Fr::load(vb + (int64_t)t * D, lg, vf);
    if (ph) Fr::rotate(ph + (int64_t)run.pl[16 * ch + lm] * (D / 2), lg, kf);
    if (d.norm) Fr::template normalise<true>(kf, d.eps);
    wave_lds_fence();  // the last chunk's reads are done
    Fr::to_lds(kt + lm * LD, lg, kf);
    if constexpr (X) to_lds16(reinterpret_cast<char*>(vt), lm, lg, vr.v);
    else Fr::to_lds(vt + lm * LD, lg, vf);
    wave_lds_fence();
    f32x4 y;
    if constexpr (X) {
      from_lds16(reinterpret_cast<const char*>(vt), m, g, vr.v);
      y = contract16(vr.v, gr.v);
    } else {
      Fr::from_lds(vt + m * LD, g, vf);
      y = contract<Fr::N>(vf, gf);
    }
    Fr::from_lds(kt + m * LD, g, kf);
    const f32x4 s = contract<Fr::N>(kf, qf);
    float ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float pw = exp_of(fmaf(s[r], d.scale, -L));
      ds[r] = pick(see, r, pw * (y[r] - Dv), 0.f);
    }
    // a row of K~ that is not finite makes every score of its row so
    const float sv[4] = {s[0], s[1], s[2], s[3]};
    if (__any(not_finite<4>(sv, 0.f) != 0.f)) {
      add_in_window<CPL, false>(acc, ds, see, m, g, [&](int j, int r, int e) { return kt[(4 * j + r) * LD + e]; });
    } else {
      float ka[4][CPL];
#pragma unroll
      for (int r = 0; r < 4; ++r) load_n<float, CPL>(kt + (4 * g + r) * LD + m * CPL, ka[r]);
      add_product<false>(acc, ka, ds);
    }
  });
  if (d.split > 1) {
    __syncthreads();
    merge_waves<CPL>(acc, lds, WAVE, wave, part, d.split, lane);
  }
  if (at.store) finish_row<T, D>(acc, d.scale, q + row * D, phq, d, g, w.live, dq + row * D);
}

// ---- dk, dv ----------------------------------------------------------------
template <typename T, int D, bool X>
__global__ void __launch_bounds__(256, D == 64 ? 3 : 1) na3d_any_dkdv_kernel(const T* __restrict__ q, const T* __restrict__ k,
                                                            const T* __restrict__ v, const float2* __restrict__ cs,
                                                            const T* __restrict__ dout, const T* __restrict__ dlo,
                                                            const float* __restrict__ lse, const float* __restrict__ dvec,
                                                            T* __restrict__ dk, T* __restrict__ dv, AnyDims d) {
  using Fr = Frag<T, D>;
  constexpr int CPL = D / 16, LD = D + 4, GT = X ? 4 * row16(D) : 16 * LD;  // floats of the dO tile
  constexpr int WAVE = 16 * LD + GT + 32;
  __shared__ __attribute__((aligned(16))) float lds[4 * WAVE];
  __shared__ __attribute__((aligned(16))) Run run;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const int lm = lane >> 2, lg = lane & 3;  // row and piece that the lane loads
  const uint32_t launched = blockIdx.y * gridDim.x + blockIdx.x;
  if (launched >= d.blocks) return;
  const Place at = wave_place(d, launched, wave);
  const int part = at.part;
  const Walk w = Walk::make<true>(d, at.tile, m);
  const int64_t n_tok = (int64_t)d.Z * d.H * d.W, base = at.bh * n_tok;
  const uint32_t mine = w.mine();
  const float2* ph = cs ? cs + (int64_t)at.b * d.H * d.W * (D / 2) : nullptr;
  const float2* phk = ph ? ph + (int64_t)w.mine_in_plane() * (D / 2) : nullptr;
  const T *qb = q + base * D, *gb = dout + base * D, *lb = dlo ? dlo + base * D : nullptr;
  const int64_t row = base + mine;
  float *qt = lds + wave * WAVE, *gt = qt + 16 * LD, *st = gt + GT;

  float kf[Fr::N], vf[Fr::N];
  Fr::load(k + row * D, g, kf);
  if (phk) Fr::rotate(phk, g, kf);
  if (d.norm) Fr::template normalise<false>(kf, d.eps);
  typename Fr::Raw vr;
  if constexpr (X) Fr::load(v + row * D, g, vr);
  else Fr::load(v + row * D, g, vf);
  f32x4 ak[CPL], av[CPL];
#pragma unroll
  for (int c = 0; c < CPL; ++c) ak[c] = av[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  walk_box(w, run, d, part, lane, [&](uint32_t ch, uint32_t see) __attribute__((always_inline)) {
    const uint32_t t = run.tok[16 * ch + lm];
    float qf[Fr::N], gf[Fr::N];
    typename Fr::Raw gr;
    Fr::load(qb + (int64_t)t * D, lg, qf);
    const float stat = lg == 0 ? lse[base + t] : lg == 1 ? dvec[base + t] : 0.f;
    if constexpr (X) {
      Fr::load(gb + (int64_t)t * D, lg, gr);
    } else {
      Fr::load(gb + (int64_t)t * D, lg, gf);
      if (lb) {
        float lf[Fr::N];
        Fr::load(lb + (int64_t)t * D, lg, lf);
#pragma unroll
        for (int i = 0; i < Fr::N; ++i) gf[i] += lf[i];
      }
    }
    if (ph) Fr::rotate(ph + (int64_t)run.pl[16 * ch + lm] * (D / 2), lg, qf);
    if (d.norm) Fr::template normalise<true>(qf, d.eps);
    wave_lds_fence();  // the last chunk's reads are done
    Fr::to_lds(qt + lm * LD, lg, qf);
    if constexpr (X) to_lds16(reinterpret_cast<char*>(gt), lm, lg, gr.v);
    else Fr::to_lds(gt + lm * LD, lg, gf);
    if (lg < 2) st[16 * lg + lm] = stat;
    wave_lds_fence();
    f32x4 y;
    if constexpr (X) {
      from_lds16(reinterpret_cast<const char*>(gt), m, g, gr.v);
      y = contract16(gr.v, vr.v);
    } else {
      Fr::from_lds(gt + m * LD, g, gf);
      y = contract<Fr::N>(gf, vf);
    }
    Fr::from_lds(qt + m * LD, g, qf);
    const f32x4 s = contract<Fr::N>(qf, kf);
    const float4 L = *reinterpret_cast<const float4*>(st + 4 * g), Dv = *reinterpret_cast<const float4*>(st + 16 + 4 * g);
    const float Ls[4] = {L.x, L.y, L.z, L.w}, Ds[4] = {Dv.x, Dv.y, Dv.z, Dv.w};
    float pw[4], ds[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      pw[r] = pick(see, r, exp_of(fmaf(s[r], d.scale, -Ls[r])), 0.f);
      ds[r] = pick(see, r, pw[r] * (y[r] - Ds[r]), 0.f);
    }
    // a row of Q~ or dO that is not finite makes every score or product of its row so
    const float sy[8] = {s[0], s[1], s[2], s[3], y[0], y[1], y[2], y[3]};
    if (__any(not_finite<8>(sy, 0.f) != 0.f)) {
      add_in_window<CPL, X>(av, pw, see, m, g, [&](int j, int r, int e) {
        if constexpr (X)
          return ldf(reinterpret_cast<const uint16_t*>(reinterpret_cast<const char*>(gt) + (4 * j + r) * row16(D)) + e);
        else
          return gt[(4 * j + r) * LD + e];
      });
      add_in_window<CPL, false>(ak, ds, see, m, g, [&](int j, int r, int e) { return qt[(4 * j + r) * LD + e]; });
    } else {
      float a[4][CPL];
      if constexpr (X) {
        add_product16<CPL>(av, reinterpret_cast<const char*>(gt), m, g, pw);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) load_n<float, CPL>(gt + (4 * g + r) * LD + m * CPL, a[r]);
        add_product<false>(av, a, pw);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) load_n<float, CPL>(qt + (4 * g + r) * LD + m * CPL, a[r]);
      add_product<false>(ak, a, ds);
    }
  });
  if (d.split > 1) {
    __syncthreads();
    merge_waves<CPL>(ak, lds, WAVE, wave, part, d.split, lane);
    __syncthreads();
    merge_waves<CPL>(av, lds, WAVE, wave, part, d.split, lane);
  }
  if (!at.store) return;
  finish_row<T, D>(ak, d.scale, k + row * D, phk, d, g, w.live, dk + row * D);
  if (w.live) {
    float o[4 * CPL];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < CPL; ++c) o[channel<CPL, X>(0, c, r)] = av[c][r];
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
  const LaunchGrid g = launch_grid(a.blocks);
  return dim3(g.x, g.y);
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
  const bool x = sizeof(T) == 2 && !o.dout_lo;
#define STRATA_ANY(K, XX, ...)                                                                                       \
  hipLaunchKernelGGL((K<T, D, XX>), any_grid(a), dim3(256), 0, s, static_cast<const T*>(q), static_cast<const T*>(k), \
                     static_cast<const T*>(v), c2, static_cast<const T*>(dout), static_cast<const T*>(o.dout_lo), lse, \
                     dvec, __VA_ARGS__, a)
  if (part == 1) {
    if (x) STRATA_ANY(na3d_any_dq_kernel, sizeof(T) == 2, static_cast<T*>(dq));
    else STRATA_ANY(na3d_any_dq_kernel, false, static_cast<T*>(dq));
  } else {
    if (x) STRATA_ANY(na3d_any_dkdv_kernel, sizeof(T) == 2, static_cast<T*>(dk), static_cast<T*>(dv));
    else STRATA_ANY(na3d_any_dkdv_kernel, false, static_cast<T*>(dk), static_cast<T*>(dv));
  }
#undef STRATA_ANY
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
