// Row pass of the attention backward with the sigmoid output gate (App. B.5):
//   D = <dO, out>, and with a = sigmoid(g):  dA = a dO,
//   dgate = (1 - a) dO out per channel, or (1 - a) D for one logit per (token,
//   head); 1 - a is evaluated as sigmoid(-g).
// dA feeds the attention backward in place of dO.  For bf16 it is written as
// two terms, hi = bf16(dA) and lo = bf16(dA - hi), whose sum carries dA to
// ~2^-16 relative: rounding dA to bf16 alone would cost more than a percent of
// the gradients' RMS.  A lane handles one 16-byte piece of a row (8 bf16 or 4
// float32 values); the CPR lanes of a row are consecutive and aligned inside
// the wave and add their partial sums by butterfly exchanges.  Arithmetic in
// float32.
#include "common.h"
#include "kernels.h"

namespace strata {
namespace {

template <typename T>
struct Piece;
template <>
struct Piece<uint16_t> {  // 8 bf16
  static constexpr int E = 8;
  static __device__ __forceinline__ void unpack(const uint4& u, float* f) {
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
    }
  }
  static __device__ __forceinline__ uint4 pack(const float* f) {
    return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                      pack_bf16x2(f[6], f[7]));
  }
  static __device__ __forceinline__ float load1(const uint16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void store1(uint16_t* p, float v) { *p = f32_to_bf16(v); }
  // remainders f - bf16(f), rounded to bf16
  static __device__ __forceinline__ uint4 pack_lo(const float* f) {
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = f[i] - bf16_to_f32(f32_to_bf16(f[i]));
    return pack(r);
  }
};
template <>
struct Piece<float> {  // 4 float32
  static constexpr int E = 4;
  static __device__ __forceinline__ void unpack(const uint4& u, float* f) {
    f[0] = __uint_as_float(u.x);
    f[1] = __uint_as_float(u.y);
    f[2] = __uint_as_float(u.z);
    f[3] = __uint_as_float(u.w);
  }
  static __device__ __forceinline__ uint4 pack(const float* f) {
    return make_uint4(__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                      __float_as_uint(f[3]));
  }
  static __device__ __forceinline__ float load1(const float* p) { return *p; }
  static __device__ __forceinline__ void store1(float* p, float v) { *p = v; }
  static __device__ __forceinline__ uint4 pack_lo(const float*) { return make_uint4(0u, 0u, 0u, 0u); }
};

__device__ __forceinline__ float sigm(float g) { return 1.f / (1.f + expf(-g)); }

template <int CPR>
__device__ __forceinline__ float row_sum(float x) {
#pragma unroll
  for (int off = CPR / 2; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

template <typename T, int D>
__global__ void __launch_bounds__(256) gate_prep_kernel(const T* __restrict__ out, const T* __restrict__ dout,
                                                        const T* __restrict__ gate, int gate_dim,
                                                        float* __restrict__ dvec, T* __restrict__ da,
                                                        T* __restrict__ da_lo, T* __restrict__ dgate, int64_t n) {
  using PC = Piece<T>;
  constexpr int E = PC::E, CPR = D / E;
  static_assert(64 % CPR == 0, "a row's lanes must not straddle a wave");
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = gid / CPR;
  const int c = (int)(gid % CPR);
  const bool live = row < n;
  float o[E], g[E];
  float acc = 0.f;
  if (live) {
    PC::unpack(*reinterpret_cast<const uint4*>(out + row * D + c * E), o);
    PC::unpack(*reinterpret_cast<const uint4*>(dout + row * D + c * E), g);
#pragma unroll
    for (int e = 0; e < E; ++e) acc = fmaf(g[e], o[e], acc);
  }
  const float Dr = row_sum<CPR>(acc);
  if (!live) return;
  if (c == 0) dvec[row] = Dr;
  if (!gate) return;
  float a[E], ra[E];  // sigmoid(g), sigmoid(-g) = 1 - sigmoid(g)
  if (gate_dim == 1) {
    const float gl = PC::load1(gate + row);
    const float s = sigm(gl), rs = sigm(-gl);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      a[e] = s;
      ra[e] = rs;
    }
    if (c == 0) PC::store1(dgate + row, rs * Dr);
  } else {
    float gl[E];
    PC::unpack(*reinterpret_cast<const uint4*>(gate + row * D + c * E), gl);
    float dg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
      a[e] = sigm(gl[e]);
      ra[e] = sigm(-gl[e]);
      dg[e] = ra[e] * g[e] * o[e];
    }
    *reinterpret_cast<uint4*>(dgate + row * D + c * E) = PC::pack(dg);
  }
  float d[E];
#pragma unroll
  for (int e = 0; e < E; ++e) d[e] = a[e] * g[e];
  *reinterpret_cast<uint4*>(da + row * D + c * E) = PC::pack(d);
  if (da_lo) *reinterpret_cast<uint4*>(da_lo + row * D + c * E) = PC::pack_lo(d);
}

// bf16 with one gate logit per (token, head).  With a = sigmoid(g) = f 2^e, f in
// [1/2, 1), the gated backward is the plain one on
//   dO' = 2^e dO (exact in bf16),  lse' = lse - ln f,  D' = D / f:
// P' = f P, so P' (dO'.v - D') = P (a dO.v - D) and P' dO' = P a dO.  No rounded
// dA is formed: the attention kernels take one bf16 tensor (as without a gate)
// instead of dA in two terms, which the balanced dK/dV kernel has no room for,
// and the range of a goes into dO' instead of P', whatever the gate.  a = 0 gives
// dO' = 0.
// The balanced kernel takes dO' and V in float16 (dO' under one scale per (batch,
// head)), a narrower range than bf16's, and a shut gate spreads dO' widely; so a
// pass over dO' and V tells it which heads fit, and the one-block kernel takes the
// others.
// Measured at 24 tiles x 16 heads x 24x16x16, 9x9x9, QK norm, the whole backward:
// 9.58 ms with dA in two terms, 7.37 ms now (8.21 ms with the one-block kernel alone);
// reading V takes 45 us of it, the one-block launch that finds every head taken 35.
using half2u = uint16_t __attribute__((ext_vector_type(2)));

// largest magnitude of a row's bf16 values as bits, from its 16-byte pieces in 2^log2_cpr lanes
__device__ __forceinline__ uint32_t row_max_bits(uint4 x, int log2_cpr) {
  auto mag = [](uint32_t w) { return __builtin_bit_cast(half2u, w & 0x7FFF7FFFu); };
  half2u m = __builtin_elementwise_max(__builtin_elementwise_max(mag(x.x), mag(x.y)),
                                       __builtin_elementwise_max(mag(x.z), mag(x.w)));
  for (int off = 1 << log2_cpr >> 1; off > 0; off >>= 1)
    m = __builtin_elementwise_max(m, __builtin_bit_cast(half2u, __shfl_xor(__builtin_bit_cast(uint32_t, m), off)));
  return max(m.x, m.y);
}

__global__ void __launch_bounds__(256) gate_row_prep_kernel(const uint16_t* __restrict__ out,
                                                            const uint16_t* __restrict__ dout,
                                                            const uint16_t* __restrict__ gate,
                                                            const float* __restrict__ lse,
                                                            const uint16_t* __restrict__ v, uint32_t* __restrict__ row_max,
                                                            float* __restrict__ lse_f,
                                                            float* __restrict__ dvec, uint16_t* __restrict__ da,
                                                            uint16_t* __restrict__ dgate, int64_t n, int log2_cpr) {
  using PC = Piece<uint16_t>;
  constexpr int E = PC::E;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t row = gid >> log2_cpr;
  const bool live = row < n;
  float o[E], g[E];
  float Dr = 0.f;
  if (live) {
    PC::unpack(*reinterpret_cast<const uint4*>(out + gid * E), o);
    PC::unpack(*reinterpret_cast<const uint4*>(dout + gid * E), g);
#pragma unroll
    for (int e = 0; e < E; ++e) Dr = fmaf(g[e], o[e], Dr);
  }
  for (int off = 1 << log2_cpr >> 1; off > 0; off >>= 1) Dr += __shfl_xor(Dr, off);
  if (!live) return;
  const float gl = PC::load1(gate + row);
  const float a = sigm(gl);
  int e2 = 0;
  float f = frexpf(a, &e2);
  float mul = ldexpf(1.f, e2);
  if (a == 0.f) {
    f = 0.5f;
    mul = 0.f;
  }
  if ((gid & ((1 << log2_cpr) - 1)) == 0) {
    PC::store1(dgate + row, sigm(-gl) * Dr);
    dvec[row] = Dr / f;
    lse_f[row] = lse[row] - logf(f);
  }
#pragma unroll
  for (int e = 0; e < E; ++e) g[e] *= mul;
  const uint4 packed = PC::pack(g);
  *reinterpret_cast<uint4*>(da + gid * E) = packed;
  if (v) {
    const uint32_t mo = row_max_bits(packed, log2_cpr);
    const uint32_t mv = row_max_bits(*reinterpret_cast<const uint4*>(v + gid * E), log2_cpr);
    if ((gid & ((1 << log2_cpr) - 1)) == 0) row_max[row] = mo | mv << 16;
  }
}

// Whether a (batch, head) fits the balanced kernel's float16 operands, from its
// rows' largest magnitudes (one workgroup per (batch, head)); a row of zeros always
// does.
//   V: below 2^16 (the largest bf16 value there is 65280), and every row's largest
//     value at least 2^-10, so that float16's spacing of 2^-24 is 2^-14 of it;
//   dO': finite, and every row's largest value within 2^24 of the head's, which is
//     staged between 2^13 and 2^14: half of 2^-24 is 2^-14 of it or less.
// 2^-14 is a quarter of the rounding of dS, and less than P had in bf16.
constexpr int kFitsThreads = 1024;
__global__ void __launch_bounds__(kFitsThreads) gate_fits_kernel(const uint32_t* __restrict__ row_max,
                                                                 int* __restrict__ fits, int64_t n) {
  const uint32_t* w = row_max + blockIdx.x * n;
  uint32_t omax = 0, omin = 0xFFFFu, vmax = 0, vmin = 0xFFFFu;
  for (int64_t i0 = threadIdx.x; i0 < n; i0 += 8 * kFitsThreads) {
    uint32_t x[8];  // loads in flight together: a head's rows are read by one workgroup
#pragma unroll
    for (int t = 0; t < 8; ++t) x[t] = w[min(i0 + t * kFitsThreads, n - 1)];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const uint32_t o = x[t] & 0xFFFFu, v = x[t] >> 16;
      omax = max(omax, o);
      vmax = max(vmax, v);
      omin = o ? min(omin, o) : omin;
      vmin = v ? min(vmin, v) : vmin;
    }
  }
  constexpr int kWaves = kFitsThreads / 64;
  __shared__ uint32_t part[kWaves][4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    omax = max(omax, (uint32_t)__shfl_xor((int)omax, off));
    omin = min(omin, (uint32_t)__shfl_xor((int)omin, off));
    vmax = max(vmax, (uint32_t)__shfl_xor((int)vmax, off));
    vmin = min(vmin, (uint32_t)__shfl_xor((int)vmin, off));
  }
  if ((threadIdx.x & 63) == 0) {
    uint32_t* p = part[threadIdx.x >> 6];
    p[0] = omax; p[1] = omin; p[2] = vmax; p[3] = vmin;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
#pragma unroll
  for (int t = 1; t < kWaves; ++t) {
    omax = max(omax, part[t][0]);
    omin = min(omin, part[t][1]);
    vmax = max(vmax, part[t][2]);
    vmin = min(vmin, part[t][3]);
  }
  constexpr uint32_t kInf = 0x7F80u, k2p16 = (127u + 16u) << 7, k2m10 = (127u - 10u) << 7;
  fits[blockIdx.x] = omax < kInf && (omin >> 7) + 24 >= omax >> 7 && vmax < k2p16 && vmin >= k2m10;
}

int64_t rows(const strata_na3d_desc& d) { return (int64_t)d.B * d.heads * d.Z * d.H * d.W; }

template <typename T, int D>
unsigned blocks_for(int64_t n) {
  constexpr int CPR = D / Piece<T>::E;
  return (unsigned)((n * CPR + 255) / 256);
}

}  // namespace

#define STRATA_DISPATCH_TD(d, F)                       \
  do {                                                 \
    if ((d).dtype == STRATA_BF16) {                    \
      if ((d).head_dim == 32) F(uint16_t, 32);         \
      else if ((d).head_dim == 64) F(uint16_t, 64);    \
      else F(uint16_t, 128);                           \
    } else {                                           \
      if ((d).head_dim == 32) F(float, 32);            \
      else if ((d).head_dim == 64) F(float, 64);       \
      else F(float, 128);                              \
    }                                                  \
  } while (0)

void launch_na3d_bwd_gate_prep(const strata_na3d_desc& d, const NaOpts& o, const void* out,
                               const void* dout, float* dvec, void* da_hi, void* da_lo, void* dgate,
                               hipStream_t s) {
  const int64_t n = rows(d);
#define F(T, D)                                                                                   \
  hipLaunchKernelGGL((gate_prep_kernel<T, D>), dim3(blocks_for<T, D>(n)), dim3(256), 0, s,        \
                     static_cast<const T*>(out), static_cast<const T*>(dout),                    \
                     static_cast<const T*>(o.gate), o.gate_dim, dvec, static_cast<T*>(da_hi),     \
                     static_cast<T*>(da_lo), static_cast<T*>(dgate), n)
  STRATA_DISPATCH_TD(d, F);
#undef F
}

void launch_na3d_bwd_gate_row_prep(const strata_na3d_desc& d, const NaOpts& o, const void* out, const void* dout,
                                   const float* lse, const void* v, float* lse_f, float* dvec, void* da, void* dgate,
                                   uint32_t* row_max, int* fits, hipStream_t s) {
  const int64_t n = rows(d);
  const int l2 = d.head_dim == 32 ? 2 : d.head_dim == 64 ? 3 : 4;  // 16-byte pieces per row
  hipLaunchKernelGGL(gate_row_prep_kernel, dim3((unsigned)(((n << l2) + 255) / 256)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(out), static_cast<const uint16_t*>(dout),
                     static_cast<const uint16_t*>(o.gate), lse, static_cast<const uint16_t*>(v), row_max, lse_f, dvec,
                     static_cast<uint16_t*>(da), static_cast<uint16_t*>(dgate), n, l2);
  if (v)
    hipLaunchKernelGGL(gate_fits_kernel, dim3((unsigned)(d.B * d.heads)), dim3(kFitsThreads), 0, s, row_max, fits,
                       (int64_t)d.Z * d.H * d.W);
}

}  // namespace strata
