// Column-wise attention for gfx950 (Sec. 3.2: attention along the vertical
// within each column, alternating with the NA3D blocks), as neighbourhood
// attention with window (kz, 1, 1): a query at level i of column (y, x) sees the
// kz levels [s, s + kz) of its own column, s = clamp(i - (kz-1)/2, 0, Z - kz);
// kz = Z is the full column.  bf16 in/out, head_dim 64, Z <= 32.
//
// StereoRoPE: every token of a column has the same (y, x) and so the same
// rotation R; <R q, R k> = <q, k>, so the rotation cancels exactly and is not
// applied (the phase table is not read).
//
// Work decomposition: one wave per (tile, head, y, x) column, grid-strided.
// The column's levels are padded to 16 NB (NB = 1 or 2 blocks of 16):
//   S^T (keys x queries) = K . Q^T   float16 MFMA 16x16x32, two per (key block,
//                                    query block); Q is scaled by scale log2(e)
//                                    (times its QK RMSNorm factor) and K by its
//                                    norm factor in float32 before the float16
//                                    rounding, both straight from global memory;
//                                    the accumulator is seeded with the window
//                                    mask (0 or -inf; padded levels -inf);
//   P = exp2(S^T - max) in one pass (all keys of a query are present), bf16;
//   O^T (64 d x 16 queries) += V^T . P^T  bf16 MFMA with the V^T fragments read
//                                    by the LDS transpose read from the column's
//                                    V rows, staged by the direct-to-LDS copy
//                                    (160-byte rows, pad columns copy column 0);
//   L = 1 . P^T                      the row sums (every lane gets its query's).
// Row m of the transposed tile t is channel 32 (t/2) + 8 (m/4) + 4 (t%2) + m%4, so
// that a lane ends with channels 8g..8g+7 and 32+8g..32+8g+7 of its token: the
// 16-byte pieces in which rows are loaded are the pieces it stores.
// The lane layouts are those of the neighbourhood kernels: a lane (qn, g) holds
// keys 16c + 4g + i of query qn in S^T, and P^T packed in place is the B operand
// of the P.V product with the keys in the same (permuted) order as the
// transpose reads deliver V.
#include "common.h"
#include "kernels.h"
#include "mfma_util.h"

namespace strata {
namespace {

using namespace mfma;

constexpr int kD = 64;
constexpr int kVRow = 160;           // LDS bytes per staged V row (8 data + 2 pad 16-byte columns)
constexpr int kWaves = 4;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// byte offset of transposed tile t inside a row (the lane adds 16 bytes per row group)
__device__ __forceinline__ constexpr int tr_col(int t) { return 64 * (t >> 1) + 8 * (t & 1); }

// two tiles (t, t + 1) of a lane's results -> 8 consecutive bf16 channels
__device__ __forceinline__ uint4 pack8(const f32x4& a, const f32x4& b) {
  return make_uint4(pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]), pack2(b[2], b[3]));
}

struct ColArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  uint16_t* out;
  float* lse;
  const uint16_t* gate;  // with GATE: logits per (token, head) (gate_dim 1) or per channel
  int gate_dim;
  float eps;
  int Z, kz;
  int64_t HW;            // tokens per level
  int64_t ncol;          // B * heads * H * W
  float qscale;          // scale * log2(e)
};

template <int NB, bool NORM, bool GATE>
__global__ void __launch_bounds__(64 * kWaves) na3d_col_kernel(ColArgs a) {
  constexpr int ZP = 16 * NB;                       // padded levels
  constexpr int SLOTS = ZP * (kVRow / 16);          // 16-byte slots of the V tile
  constexpr int ITV = (SLOTS + 63) / 64;            // copy instructions per wave
  __shared__ __attribute__((aligned(16))) char sV[kWaves][ITV * 64 * 16];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, qn = lane & 15;
  const int Z = a.Z, kz = a.kz;
  const int64_t HW = a.HW;
  char* tv = sV[wave];

  // lane-constant parts: V copy offsets (rows clamped into the column, pad
  // columns copy column 0) and transpose-read addresses
  int vrow[ITV], vcol[ITV];  // level and element offset in the row of this lane's V slots
#pragma unroll
  for (int it = 0; it < ITV; ++it) {
    const int s = it * 64 + lane;
    vrow[it] = min(min(s / 10, ZP - 1), Z - 1);
    vcol[it] = (s % 10 < 8 ? s % 10 : 0) * 8;
  }
  uint32_t vaddr[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) vaddr[c] = (16 * c + 4 * g + (qn >> 2)) * kVRow + (qn & 3) * 16;
  // window mask, per (query block, key block): key 16c + 4g + i of query 16b + qn
  f32x4 bias[NB][NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int qi = min(16 * b + qn, Z - 1);
    const int ws = win_start(qi, Z, kz);
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int j = 16 * c + 4 * g + i;
        bias[b][c][i] = (j < Z && j >= ws && j < ws + kz) ? 0.f : -INFINITY;
      }
  }
  const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));

  const int64_t nwaves = (int64_t)gridDim.x * kWaves;
  for (int64_t col = (int64_t)blockIdx.x * kWaves + wave; col < a.ncol; col += nwaves) {
    // column (t, h, y, x) = col: token of level z is ((t*heads + h) * Z + z) * HW + yx
    const int64_t th = col / HW, yx = col - th * HW;
    const int64_t base = th * Z * HW + yx;  // token index of level 0
    auto tok = [&](int z) { return base + (int64_t)z * HW; };

    // V rows -> LDS (direct copy); its wait comes before the transpose reads
#pragma unroll
    for (int it = 0; it < ITV; ++it) copy16_to_lds(a.v + tok(vrow[it]) * kD + vcol[it], tv + it * 64 * 16);
    // Q (B operand) and K (A operand) fragments: level 16b + qn, d = 8g.. and 32 + 8g..
    uint4 qraw[NB][2], kraw[NB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int z = min(16 * b + qn, Z - 1);
      const uint4* qs = reinterpret_cast<const uint4*>(a.q + tok(z) * kD);
      const uint4* ks = reinterpret_cast<const uint4*>(a.k + tok(z) * kD);
      qraw[b][0] = qs[g];
      qraw[b][1] = qs[4 + g];
      kraw[b][0] = ks[g];
      kraw[b][1] = ks[4 + g];
    }
    f16x8 qf[NB][2], kf[NB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float mq = a.qscale, mk = 1.f;
      if constexpr (NORM) {  // the 4 lanes of a row hold its 64 values
        mq *= __builtin_amdgcn_rsqf(sum_over_rows(sumsq8(qraw[b][1], sumsq8(qraw[b][0], 0.f))) * (1.f / kD) + a.eps);
        mk = __builtin_amdgcn_rsqf(sum_over_rows(sumsq8(kraw[b][1], sumsq8(kraw[b][0], 0.f))) * (1.f / kD) + a.eps);
      }
      qf[b][0] = __builtin_bit_cast(f16x8, scale8h(qraw[b][0], mq));
      qf[b][1] = __builtin_bit_cast(f16x8, scale8h(qraw[b][1], mq));
      kf[b][0] = __builtin_bit_cast(f16x8, scale8h(kraw[b][0], mk));
      kf[b][1] = __builtin_bit_cast(f16x8, scale8h(kraw[b][1], mk));
    }
    __builtin_amdgcn_s_waitcnt(0);  // this lane's V copies have landed (each lane reads its own wave's tile)
    __builtin_amdgcn_wave_barrier();
    // V^T fragments: d block t, keys of chunks (0, 1)
    bf16x8 vf[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const i16x4 lo = tr_read(tv + vaddr[0] + tr_col(t));
      const i16x4 hi = NB > 1 ? tr_read(tv + vaddr[NB > 1 ? 1 : 0] + tr_col(t)) : i16x4{0, 0, 0, 0};
      const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
      vf[t] = __builtin_bit_cast(bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
    }

#pragma unroll
    for (int b = 0; b < NB; ++b) {  // query block
      f32x4 s[NB];
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        const f32x4 acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[c][0], qf[b][0], bias[b][c], 0, 0, 0);
        s[c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[c][1], qf[b][1], acc, 0, 0, 0);
      }
      float mx = fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3]));
      if constexpr (NB > 1) mx = fmaxf(mx, fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
      mx = max_over_rows(mx);
      uint32_t pk[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        pk[c][0] = pack2(__builtin_amdgcn_exp2f(s[c][0] - mx), __builtin_amdgcn_exp2f(s[c][1] - mx));
        pk[c][1] = pack2(__builtin_amdgcn_exp2f(s[c][2] - mx), __builtin_amdgcn_exp2f(s[c][3] - mx));
      }
      const bf16x8 pf = __builtin_bit_cast(bf16x8, make_uint4(pk[0][0], pk[0][1], pk[1][0], pk[1][1]));
      f32x4 o[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        o[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[t], pf, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      const f32x4 lsum = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      const int z = 16 * b + qn;
      if (z < Z) {
        const float lt = lsum[0];
        float inv = 1.f / lt;
        const int64_t tk = tok(z);
        if constexpr (GATE)
          if (a.gate_dim == 1) inv *= sigmoid_fast(bf16_to_f32(a.gate[tk]));
        uint4* dst = reinterpret_cast<uint4*>(a.out + tk * kD);
        f32x4 r[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) r[t] = o[t] * inv;
        if constexpr (GATE)
          if (a.gate_dim != 1) {
            const uint4* gs = reinterpret_cast<const uint4*>(a.gate + tk * kD);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const uint4 w = gs[4 * h + g];
              r[2 * h] *= sigmoid4_bf16(make_uint2(w.x, w.y));
              r[2 * h + 1] *= sigmoid4_bf16(make_uint2(w.z, w.w));
            }
          }
        dst[g] = pack8(r[0], r[1]);
        dst[4 + g] = pack8(r[2], r[3]);
        if (a.lse && g == 0) a.lse[tk] = (mx + __log2f(lt)) * kLn2;
      }
    }
    __builtin_amdgcn_wave_barrier();  // the next column's copies overwrite this wave's V tile
  }
}

}  // namespace

// Column-wise forward for windows (kz, 1, 1) with Z <= 32 (bf16, head_dim 64);
// false for any other problem.
bool launch_na3d_fwd_col(const strata_na3d_desc& d, const NaOpts& o, const void* q, const void* k,
                         const void* v, void* out, float* lse, hipStream_t s) {
  if (d.dtype != STRATA_BF16 || d.head_dim != kD || d.ky != 1 || d.kx != 1 || d.Z > 32) return false;
  ColArgs a = {};
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.gate = static_cast<const uint16_t*>(o.gate);
  a.gate_dim = o.gate_dim;
  a.eps = o.eps;
  a.Z = d.Z;
  a.kz = d.kz;
  a.HW = (int64_t)d.H * d.W;
  a.ncol = (int64_t)d.B * d.heads * a.HW;
  a.qscale = d.scale * kLog2e;
  const int64_t want = (a.ncol + kWaves - 1) / kWaves;
  const unsigned blocks = (unsigned)(want < 65536 ? want : 65536);
  const dim3 grid(blocks), block(64 * kWaves);
  const bool nb2 = d.Z > 16;
#define L(NB, N, G) hipLaunchKernelGGL((na3d_col_kernel<NB, N, G>), grid, block, 0, s, a)
  if (nb2) {
    if (o.qk_norm) { if (o.gate) L(2, true, true); else L(2, true, false); }
    else { if (o.gate) L(2, false, true); else L(2, false, false); }
  } else {
    if (o.qk_norm) { if (o.gate) L(1, true, true); else L(1, true, false); }
    else { if (o.gate) L(1, false, true); else L(1, false, false); }
  }
#undef L
  return true;
}

// ---------------------------------------------------------------------------
// Column-wise attention backward: dq, dk, dv (and dgate) of one column per wave,
// in one pass over q, k, v, out, dO and the gate.
//
// A lane's fragments of a row (level 16b + qn, d = 8g.. and 32 + 8g..) serve as
// the A operand and as the B operand of a 16x16x32 MFMA alike, so both
// orientations come from the same registers:
//   queries as columns (dq):  S^T = K^ Q^T seeded with the mask, P^T = exp2(S^T
//     - lse2), Y^T = V dO^T - D, dS^T = P^T Y^T, dQ^T = K^T dS^T with the K^T
//     fragments read transposed from the float16 K^ rows staged in LDS;
//   keys as columns (dk, dv):  S = Q K^T, P, Y = dO V^T - D, dS = P Y,
//     dV^T = dO^T P (dO rows staged in LDS), dK^T = Q^T dS (float16 Q^ rows,
//     staged where the K^ rows were).
// dS enters its float16 MFMA scaled by 2^(15 - E), E the exponent of the
// largest |dS| of the column's query (resp. key): all keys of a query are
// present at once, so one exact power-of-two scale suffices.  lse2 = lse log2 e
// and D of padded levels are +inf and 0, so their P and dS vanish.
// The forward's output is read for D = <dO, out>, so no pass of its own forms D.
// Options: QK RMSNorm (q^ = r q, k^ = r k in float32 before the float16
// rounding; dq = r (dq^ - q^ mean(dq^ q^)) and likewise dk, in float32 from the
// raw rows in registers); the gate, a = sigmoid(g):
//   one logit per token (ROW): the plain backward with lse2 - log2(a) and D / a
//     (P a dO and P (a dO.v - D) come out; a = 0: lse2 = +inf, D = 0);
//   one per channel (CHAN): dA = a dO as two bf16 terms, formed in registers.
// What bounds it: HBM (8 rows of 128 bytes read or written per token), as long as
// enough waves are resident: 9.3 KB of LDS and at most 168 registers per wave keep
// three per SIMD (more with Z <= 16).  Two blocks of levels with a gate per channel
// stage a third tile (14 KB) and have two.  Measured at 24 tiles x 16 heads x
// 24x16x16, window 24x1x1, QK norm and a gate logit per token: 0.50 ms (4.9 TB/s,
// the rate of a large copy on the card), against 0.65 ms behind a 0.15 ms pass that
// formed D and the gate's part, with one wave per SIMD or two.  (That variant, at
// 168 registers, keeps one of them in scratch.)
struct ColBwdArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* out;
  const uint16_t* dout;
  const uint16_t* gate;
  const float* lse;   // natural log
  uint16_t* dq;
  uint16_t* dk;
  uint16_t* dv;
  uint16_t* dgate;
  float eps;
  int Z, kz;
  int64_t HW, ncol;
  float scale, qscale;
};

namespace {

constexpr int kMinExp = -100;
enum { kNoGate = 0, kRowGate = 1, kChanGate = 2 };

// logistic sigmoid, correctly scaled at both ends
__device__ __forceinline__ float sigm(float g) { return 1.f / (1.f + expf(-g)); }

// dot product of 8 bf16 pairs, added to acc (the products are exact in float32)
__device__ __forceinline__ float dot8(uint4 x, uint4 y, float acc) {
  const uint32_t a[4] = {x.x, x.y, x.z, x.w}, b[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
  for (int t = 0; t < 4; ++t)
    acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a[t]), __builtin_bit_cast(bf16x2, b[t]), acc, false);
  return acc;
}

template <int NB, bool NORM, int GATE>
__global__ void __launch_bounds__(64 * kWaves, NB == 1 || GATE != kChanGate ? 3 : 2) na3d_col_bwd_kernel(ColBwdArgs a) {
  constexpr bool LO = GATE == kChanGate;
  constexpr int ZP = 16 * NB;
  constexpr int RB = 144;                            // LDS bytes per staged row
  __shared__ __attribute__((aligned(16))) char sX[kWaves][ZP * RB];             // K^, then Q^
  __shared__ __attribute__((aligned(16))) char sG[kWaves][(LO ? 2 : 1) * ZP * RB];  // dO (dA: hi, lo)
  __shared__ __attribute__((aligned(16))) float sL[kWaves][ZP];
  __shared__ __attribute__((aligned(16))) float sD[kWaves][ZP];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, qn = lane & 15;
  const int Z = a.Z, kz = a.kz;
  const int64_t HW = a.HW;
  char* tx = sX[wave];
  char* tg = sG[wave];

  // transpose-read rows of chunk c: 16c + 4g + qn/4, 8 bytes of the 16 at qn % 4
  uint32_t taddr[NB];
#pragma unroll
  for (int c = 0; c < NB; ++c) taddr[c] = (16 * c + 4 * g + (qn >> 2)) * RB + (qn & 3) * 16;
  // window bits 4 (NB b + c) + i: queries as columns (key 16c + 4g + i, query
  // 16b + qn) and keys as columns (query 16b + 4g + i, key 16c + qn)
  uint32_t bitsT = 0, bitsN = 0;
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t bit = 1u << (4 * (NB * b + c) + i);
        {
          const int qi = min(16 * b + qn, Z - 1), j = 16 * c + 4 * g + i, ws = win_start(qi, Z, kz);
          if (j < Z && j >= ws && j < ws + kz) bitsT |= bit;
        }
        {
          const int qi = min(16 * b + 4 * g + i, Z - 1), j = 16 * c + qn, ws = win_start(qi, Z, kz);
          if (j < Z && j >= ws && j < ws + kz) bitsN |= bit;
        }
      }
  // accumulator seeds 0 / -inf of a 16 x 16 block from its four bits
  auto seed = [](uint32_t bits, int first) __attribute__((always_inline)) {
    f32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      r[i] = __uint_as_float(~(uint32_t)__builtin_amdgcn_sbfe((int)bits, first + i, 1) & 0xff800000u);
    return r;
  };
  auto tr8 = [&](const char* tile, int t) {  // 16 d x 32 rows (chunks 0 and 1), transposed
    const i16x4 lo = tr_read(tile + taddr[0] + tr_col(t));
    const i16x4 hi = NB > 1 ? tr_read(tile + taddr[NB > 1 ? 1 : 0] + tr_col(t)) : i16x4{0, 0, 0, 0};
    const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
    return make_uint4(l2.x, l2.y, h2.x, h2.y);
  };
  auto dmax = [](const f32x4& x, float m) {
    return fmaxf(m, fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3]))));
  };
  auto fence = [] {  // the wave's LDS writes before, its reads after (and the reverse)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  };
  // gradient of x^ = r x carried to x (the norm's Jacobian) and stored; raw: the row's pieces
  auto store_norm = [&](f32x4 (&x)[4], const uint4 (&raw)[2], float r, bool live, uint16_t* dst)
                        __attribute__((always_inline)) {
    if constexpr (NORM) {
      uint32_t w[8] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w, raw[1].x, raw[1].y, raw[1].z, raw[1].w};
      // (through an empty asm: the float32 values of the row are formed again, not kept since it was staged)
#pragma unroll
      for (int t = 0; t < 8; ++t) asm volatile("" : "+v"(w[t]));
      f32x4 xh[4];
      float cdot = 0.f;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        xh[t] = f32x4{lo_bf16(w[2 * t]), hi_bf16(w[2 * t]), lo_bf16(w[2 * t + 1]), hi_bf16(w[2 * t + 1])} * r;
#pragma unroll
        for (int i = 0; i < 4; ++i) cdot = fmaf(x[t][i], xh[t][i], cdot);
      }
      cdot = sum_over_rows(cdot) * (1.f / kD);
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) x[t][i] = r * fmaf(-xh[t][i], cdot, x[t][i]);
    }
    if (live) {
      uint4* p = reinterpret_cast<uint4*>(dst);
      p[g] = pack8(x[0], x[1]);
      p[4 + g] = pack8(x[2], x[3]);
    }
  };

  const int64_t nwaves = (int64_t)gridDim.x * kWaves;
  for (int64_t col = (int64_t)blockIdx.x * kWaves + wave; col < a.ncol; col += nwaves) {
    const int64_t th = col / HW, yx = col - th * HW;
    const int64_t base = th * Z * HW + yx;
    auto tok = [&](int z) { return base + (int64_t)z * HW; };

    // through an empty asm per column, so that the seeds are derived where they
    // are used and not hoisted into registers
    uint32_t bT = bitsT, bN = bitsN;
    asm volatile("" : "+v"(bT), "+v"(bN));
    uint4 qr[NB][2], kr[NB][2], vr[NB][2], gr[NB][2], orow[NB][2], glr[LO ? NB : 1][2];
    float lseA[NB], dA[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int64_t tz = tok(min(16 * b + qn, Z - 1));
      auto row = [&](const uint16_t* p, uint4 (&r)[2]) {
        const uint4* s = reinterpret_cast<const uint4*>(p + tz * kD);
        r[0] = s[g];
        r[1] = s[4 + g];
      };
      row(a.dout, gr[b]);
      row(a.out, orow[b]);
      row(a.k, kr[b]);
      row(a.q, qr[b]);
      row(a.v, vr[b]);
      lseA[b] = a.lse[tz] * kLog2e;
    }
    // D, the gate, the dO rows staged
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const bool live = 16 * b + qn < Z;
      const int64_t tz = tok(min(16 * b + qn, Z - 1));
      float dj = sum_over_rows(dot8(orow[b][1], gr[b][1], dot8(orow[b][0], gr[b][0], 0.f)));
      if constexpr (GATE == kRowGate) {
        const float gl = bf16_to_f32(a.gate[tz]);
        const float s = sigm(gl);
        if (live && g == 0) a.dgate[tz] = f32_to_bf16(sigm(-gl) * dj);
        lseA[b] -= __log2f(s);             // +inf where the sigmoid is 0
        dj = s > 0.f ? dj / s : dj * 0.f;
      }
      if constexpr (GATE == kChanGate) {
        const uint4* gs = reinterpret_cast<const uint4*>(a.gate + tz * kD);
        uint4* ds = reinterpret_cast<uint4*>(a.dgate + tz * kD);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint4 gw = gs[4 * h + g];
          const uint32_t w[4] = {gw.x, gw.y, gw.z, gw.w};
          const uint32_t o[4] = {orow[b][h].x, orow[b][h].y, orow[b][h].z, orow[b][h].w};
          const uint32_t d[4] = {gr[b][h].x, gr[b][h].y, gr[b][h].z, gr[b][h].w};
          uint32_t hi[4], lo[4], dg[4];
#pragma unroll
          for (int t = 0; t < 4; ++t) {
            const float g0 = lo_bf16(w[t]), g1 = hi_bf16(w[t]), d0 = lo_bf16(d[t]), d1 = hi_bf16(d[t]);
            dg[t] = pack2(sigm(-g0) * d0 * lo_bf16(o[t]), sigm(-g1) * d1 * hi_bf16(o[t]));
            const float x0 = sigm(g0) * d0, x1 = sigm(g1) * d1;
            hi[t] = pack2(x0, x1);
            lo[t] = pack2(x0 - lo_bf16(hi[t]), x1 - hi_bf16(hi[t]));
          }
          if (live) ds[4 * h + g] = make_uint4(dg[0], dg[1], dg[2], dg[3]);
          gr[b][h] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
          glr[b][h] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        }
      }
      lseA[b] = live ? lseA[b] : INFINITY;
      dA[b] = live ? dj : 0.f;
      char* row = tg + (16 * b + qn) * RB + 16 * g;
      st16(row, gr[b][0]);
      st16(row + 64, gr[b][1]);
      if constexpr (LO) {
        st16(row + ZP * RB, glr[b][0]);
        st16(row + ZP * RB + 64, glr[b][1]);
      }
      if (g == 0) {
        sL[wave][16 * b + qn] = lseA[b];
        sD[wave][16 * b + qn] = dA[b];
      }
    }
    // norms, float16 operands, the K^ rows staged
    f16x8 kf[NB][2];
    float rq[NB], rk[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      rq[b] = 1.f;
      rk[b] = 1.f;
      if constexpr (NORM) {
        rq[b] = __builtin_amdgcn_rsqf(sum_over_rows(sumsq8(qr[b][1], sumsq8(qr[b][0], 0.f))) * (1.f / kD) + a.eps);
        rk[b] = __builtin_amdgcn_rsqf(sum_over_rows(sumsq8(kr[b][1], sumsq8(kr[b][0], 0.f))) * (1.f / kD) + a.eps);
      }
      char* row = tx + (16 * b + qn) * RB + 16 * g;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint4 k8 = scale8h(kr[b][h], rk[b]);
        kf[b][h] = __builtin_bit_cast(f16x8, k8);
        st16(row + 64 * h, k8);
      }
    }
    fence();
    // the float16 queries are formed from the raw rows in each of the two parts
    // (the factor goes through an empty asm): the first part has no registers for both
    auto queries = [&](int b, f16x8 (&f)[2]) __attribute__((always_inline)) {
      float mq = a.qscale * rq[b];
      asm volatile("" : "+v"(mq));
      f[0] = __builtin_bit_cast(f16x8, scale8h(qr[b][0], mq));
      f[1] = __builtin_bit_cast(f16x8, scale8h(qr[b][1], mq));
    };

    // ---- queries as columns: dq ----------------------------------------------
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      f32x4 ds[NB];
      f16x8 qb[2];
      queries(b, qb);
      float mx = 0.f;
      const f32x4 nd = {-dA[b], -dA[b], -dA[b], -dA[b]};
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        f32x4 s = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[c][0], qb[0], seed(bT, 4 * (NB * b + c)), 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[c][1], qb[1], s, 0, 0, 0);
        f32x4 y = nd;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vr[c][h]),
                                                      __builtin_bit_cast(bf16x8, gr[b][h]), y, 0, 0, 0);
          if constexpr (LO)
            y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vr[c][h]),
                                                        __builtin_bit_cast(bf16x8, glr[b][h]), y, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) ds[c][i] = __builtin_amdgcn_exp2f(s[i] - lseA[b]) * y[i];
        mx = dmax(ds[c], mx);
      }
      const int e = max(__builtin_amdgcn_frexp_expf(max_over_rows(mx)), kMinExp);
      const float up = __builtin_amdgcn_ldexpf(1.f, 15 - e);
      uint32_t dk2[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
      for (int c = 0; c < NB; ++c) {
        dk2[c][0] = pack2h_rne(ds[c][0] * up, ds[c][1] * up);
        dk2[c][1] = pack2h_rne(ds[c][2] * up, ds[c][3] * up);
      }
      const f16x8 df = __builtin_bit_cast(f16x8, make_uint4(dk2[0][0], dk2[0][1], dk2[1][0], dk2[1][1]));
      const float down = a.scale * __builtin_amdgcn_ldexpf(1.f, e - 15);
      f32x4 x[4];
#pragma unroll
      for (int t = 0; t < 4; ++t)
        x[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, tr8(tx, t)), df,
                                                      f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0) * down;
      const int z = 16 * b + qn;
      store_norm(x, qr[b], rq[b], z < Z, a.dq + tok(min(z, Z - 1)) * kD);
      __builtin_amdgcn_sched_barrier(0);  // one block's registers at a time
    }

    // ---- keys as columns: dk, dv ----------------------------------------------
    fence();
    f16x8 qf[NB][2];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      queries(b, qf[b]);
      char* row = tx + (16 * b + qn) * RB + 16 * g;
      st16(row, scale8h(qr[b][0], rq[b]));
      st16(row + 64, scale8h(qr[b][1], rq[b]));
    }
    fence();
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      f32x4 ds[NB];
      uint32_t pb[2][2] = {{0u, 0u}, {0u, 0u}};
      float mx = 0.f;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        const float4 l4 = *reinterpret_cast<const float4*>(&sL[wave][16 * b + 4 * g]);
        const float4 d4 = *reinterpret_cast<const float4*>(&sD[wave][16 * b + 4 * g]);
        f32x4 s = __builtin_amdgcn_mfma_f32_16x16x32_f16(qf[b][0], kf[c][0], seed(bN, 4 * (NB * b + c)), 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x32_f16(qf[b][1], kf[c][1], s, 0, 0, 0);
        f32x4 y = {-d4.x, -d4.y, -d4.z, -d4.w};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, gr[b][h]),
                                                      __builtin_bit_cast(bf16x8, vr[c][h]), y, 0, 0, 0);
          if constexpr (LO)
            y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, glr[b][h]),
                                                        __builtin_bit_cast(bf16x8, vr[c][h]), y, 0, 0, 0);
        }
        const float p0 = __builtin_amdgcn_exp2f(s[0] - l4.x), p1 = __builtin_amdgcn_exp2f(s[1] - l4.y);
        const float p2 = __builtin_amdgcn_exp2f(s[2] - l4.z), p3 = __builtin_amdgcn_exp2f(s[3] - l4.w);
        pb[b][0] = pack2(p0, p1);
        pb[b][1] = pack2(p2, p3);
        ds[b] = f32x4{p0 * y[0], p1 * y[1], p2 * y[2], p3 * y[3]};
        mx = dmax(ds[b], mx);
      }
      const int e = max(__builtin_amdgcn_frexp_expf(max_over_rows(mx)), kMinExp);
      const float up = __builtin_amdgcn_ldexpf(1.f, 15 - e);
      uint32_t db[2][2] = {{0u, 0u}, {0u, 0u}};
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        db[b][0] = pack2h_rne(ds[b][0] * up, ds[b][1] * up);
        db[b][1] = pack2h_rne(ds[b][2] * up, ds[b][3] * up);
      }
      const bf16x8 pf = __builtin_bit_cast(bf16x8, make_uint4(pb[0][0], pb[0][1], pb[1][0], pb[1][1]));
      const f16x8 df = __builtin_bit_cast(f16x8, make_uint4(db[0][0], db[0][1], db[1][0], db[1][1]));
      const float down = a.scale * __builtin_amdgcn_ldexpf(1.f, e - 15);
      f32x4 xv[4], xk[4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        xv[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, tr8(tg, t)), pf,
                                                       f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
        if constexpr (LO)
          xv[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, tr8(tg + ZP * RB, t)), pf, xv[t],
                                                         0, 0, 0);
        xk[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, tr8(tx, t)), df,
                                                       f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0) * down;
      }
      const int z = 16 * c + qn;
      const int64_t tz = tok(min(z, Z - 1));
      store_norm(xk, kr[c], rk[c], z < Z, a.dk + tz * kD);
      if (z < Z) {
        uint4* dvd = reinterpret_cast<uint4*>(a.dv + tz * kD);
        dvd[g] = pack8(xv[0], xv[1]);
        dvd[4 + g] = pack8(xv[2], xv[3]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    fence();  // LDS reads of this column precede the next column's writes
  }
}

}  // namespace

// Column-wise backward (dq, dk, dv, dgate in one pass) for windows (kz, 1, 1)
// with Z <= 32 (bf16, head_dim 64); forms D and the gate's part itself.  False
// for any other problem.
bool launch_na3d_bwd_col(const strata_na3d_desc& d, const NaOpts& o, const void* q, const void* k, const void* v,
                         const void* out, const void* dout, const float* lse, void* dq, void* dk, void* dv,
                         void* dgate, hipStream_t s) {
  if (d.dtype != STRATA_BF16 || d.head_dim != kD || d.ky != 1 || d.kx != 1 || d.Z > 32) return false;
  ColBwdArgs a = {};
  a.q = static_cast<const uint16_t*>(q);
  a.k = static_cast<const uint16_t*>(k);
  a.v = static_cast<const uint16_t*>(v);
  a.out = static_cast<const uint16_t*>(out);
  a.dout = static_cast<const uint16_t*>(dout);
  a.gate = static_cast<const uint16_t*>(o.gate);
  a.lse = lse;
  a.dq = static_cast<uint16_t*>(dq);
  a.dk = static_cast<uint16_t*>(dk);
  a.dv = static_cast<uint16_t*>(dv);
  a.dgate = static_cast<uint16_t*>(dgate);
  a.eps = o.eps;
  a.Z = d.Z;
  a.kz = d.kz;
  a.HW = (int64_t)d.H * d.W;
  a.ncol = (int64_t)d.B * d.heads * a.HW;
  a.scale = d.scale;
  a.qscale = d.scale * kLog2e;
  const int64_t want = (a.ncol + kWaves - 1) / kWaves;
  const dim3 grid((unsigned)(want < 65536 ? want : 65536)), block(64 * kWaves);
  const bool nb2 = d.Z > 16, norm = o.qk_norm != 0;
#define L(NB, N, G) hipLaunchKernelGGL((na3d_col_bwd_kernel<NB, N, G>), grid, block, 0, s, a)
#define LG(NB, N)                                   \
  do {                                              \
    if (!o.gate) L(NB, N, kNoGate);                 \
    else if (o.gate_dim == 1) L(NB, N, kRowGate);   \
    else L(NB, N, kChanGate);                       \
  } while (0)
  if (nb2) {
    if (norm) LG(2, true); else LG(2, false);
  } else {
    if (norm) LG(1, true); else LG(1, false);
  }
#undef LG
#undef L
  return true;
}

}  // namespace strata
