// Small device helpers: bf16 storage, 16-byte vector access, wavefront reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gco {

typedef uint16_t bf16_t;

__device__ __forceinline__ float bf16_to_f32(bf16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// Round to nearest, ties to even (IEEE 754 roundTiesToEven on the upper 16 bits).
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  const __bf16 b = static_cast<__bf16>(f);  // round to nearest even (v_cvt_pk_bf16_f32)
  bf16_t u;
  __builtin_memcpy(&u, &b, 2);
  return u;
}

// Two fp32 values rounded to bf16 in one word (a in the lower half).
__device__ __forceinline__ uint32_t f32x2_to_bf16x2(float a, float b) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {a, b};
  const bf16x2_t r = __builtin_convertvector(v, bf16x2_t);
  uint32_t u;
  __builtin_memcpy(&u, &r, 4);
  return u;
}

// max(x, 0) on two packed bf16 values: a negative bf16 is a negative 16-bit integer.
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t u) {
  typedef short i16x2_t __attribute__((ext_vector_type(2)));
  i16x2_t s;
  __builtin_memcpy(&s, &u, 4);
  const i16x2_t zero = {0, 0};
  s = __builtin_elementwise_max(s, zero);
  __builtin_memcpy(&u, &s, 4);
  return u;
}

// Storage traits: how a feature row is kept in HBM.
template <typename T>
struct Store;

template <>
struct Store<float> {
  static constexpr int VEC = 4;  // elements per 16-byte access
  static __device__ __forceinline__ void load(const float* p, float (&v)[4]) {
    const float4 x = *reinterpret_cast<const float4*>(p);
    v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
  }
  static __device__ __forceinline__ void store(float* p, const float (&v)[4]) {
    *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  }
  static __device__ __forceinline__ float get(const float* p) { return *p; }
  static __device__ __forceinline__ void put(float* p, float x) { *p = x; }
  static __device__ __forceinline__ float as_stored(float x) { return x; }
};

template <>
struct Store<bf16_t> {
  static constexpr int VEC = 8;
  static __device__ __forceinline__ void load(const bf16_t* p, float (&v)[8]) {
    const uint4 x = *reinterpret_cast<const uint4*>(p);
    v[0] = __uint_as_float(x.x << 16); v[1] = __uint_as_float(x.x & 0xffff0000u);
    v[2] = __uint_as_float(x.y << 16); v[3] = __uint_as_float(x.y & 0xffff0000u);
    v[4] = __uint_as_float(x.z << 16); v[5] = __uint_as_float(x.z & 0xffff0000u);
    v[6] = __uint_as_float(x.w << 16); v[7] = __uint_as_float(x.w & 0xffff0000u);
  }
  static __device__ __forceinline__ void store(bf16_t* p, const float (&v)[8]) {
    uint4 x;
    x.x = f32x2_to_bf16x2(v[0], v[1]);
    x.y = f32x2_to_bf16x2(v[2], v[3]);
    x.z = f32x2_to_bf16x2(v[4], v[5]);
    x.w = f32x2_to_bf16x2(v[6], v[7]);
    *reinterpret_cast<uint4*>(p) = x;
  }
  static __device__ __forceinline__ float get(const bf16_t* p) { return bf16_to_f32(*p); }
  static __device__ __forceinline__ void put(bf16_t* p, float x) { *p = f32_to_bf16(x); }
  static __device__ __forceinline__ float as_stored(float x) { return bf16_to_f32(f32_to_bf16(x)); }
};

// Between LDS writes of some lanes of a wavefront and LDS reads of the same locations by
// other lanes of that wavefront: the hardware executes a wavefront's LDS operations in
// program order, so no instruction is needed, but the compiler has to be told that the
// lanes communicate (otherwise it may forward a lane's own earlier store to its load).
__device__ __forceinline__ void wave_lds_handoff() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Square root of x in [2^-100, 2^100] and quotient for a denominator in [2^-30, 2^60], correctly rounded, in
// 6 and 8 instructions (of which one each at a quarter of the rate) where sqrtf() and the division take 17
// and 11 for the ranges beyond.
// sqrt: s = x rsq(x), within two ulps, corrected by its exact residual; equal to sqrtf() for every mantissa
// of both parities of the exponent, all of which were tried.  Quotient: the reciprocal after one Newton step,
// then two corrections by the exact residual: the first leaves the quotient within an ulp, after which the
// second rounds correctly (Markstein, "Computation of elementary functions on the IBM RISC System/6000
// processor", 1990); tiny quotients (below 2^-70), whose residual is no longer exact, may be an ulp off.
__device__ __forceinline__ float sqrt_in_range(float x) {
  const float y = __builtin_amdgcn_rsqf(x), s = x * y, h = 0.5f * y;
  return fmaf(fmaf(-s, s, x), h, s);
}
__device__ __forceinline__ float quotient_in_range(float n, float d) {
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.f), r, r);
  float q = n * r;
  q = fmaf(fmaf(-d, q, n), r, q);
  return fmaf(fmaf(-d, q, n), r, q);
}

// One Adam step on N embedding values, or on one weight (constants of AdamStep), with the correctly
// rounded square root and division: every launch that may update a parameter in fp32 takes the
// same step, and a subgraph does not train differently because other kernels were chosen for it.
// With a usual eps, v is taken as at least 2^-100 for its square root, 2^-50, which eps swallows: the same
// sum.  Beyond the ranges (uniform over the wavefront) the general functions serve.
template <class Step>
__device__ __forceinline__ bool adam_in_range(const Step& ad, float largest_v) {
  return ad.eps >= 1e-9f && ad.eps <= 1.f && ad.inv_sqrt_bc2 <= 64.f && !__any(largest_v > 0x1p100f);
}
template <int N, class Step>
__device__ __forceinline__ void adam_values(const Step& ad, const float (&g)[N], float (&e)[N], float (&m)[N],
                                            float (&v)[N]) {
  float top = 0.f;
#pragma unroll
  for (int x = 0; x < N; ++x) {
    m[x] = ad.b1 * m[x] + (1.f - ad.b1) * g[x];
    v[x] = ad.b2 * v[x] + (1.f - ad.b2) * g[x] * g[x];
    top = fmaxf(top, v[x]);
  }
  if (adam_in_range(ad, top)) {
#pragma unroll
    for (int x = 0; x < N; ++x) {
      const float root = sqrt_in_range(fmaxf(v[x], 0x1p-100f));
      e[x] -= ad.lr * quotient_in_range(m[x] * ad.inv_bc1, root * ad.inv_sqrt_bc2 + ad.eps);
    }
  } else {
#pragma unroll
    for (int x = 0; x < N; ++x) e[x] -= ad.lr * ((m[x] * ad.inv_bc1) / (sqrtf(v[x]) * ad.inv_sqrt_bc2 + ad.eps));
  }
}
template <class Step>
__device__ __forceinline__ void adam_value(const Step& ad, float g, float& e, float& m, float& v) {
  float g1[1] = {g}, e1[1] = {e}, m1[1] = {m}, v1[1] = {v};
  adam_values<1>(ad, g1, e1, m1, v1);
  e = e1[0];
  m = m1[0];
  v = v1[0];
}
template <class Step>
__device__ __forceinline__ void adam_weight(const Step& ad, float g, float& w, float& m, float& v) {
  m = ad.b1 * m + (1.f - ad.b1) * g;
  v = ad.b2 * v + (1.f - ad.b2) * g * g;
  if (adam_in_range(ad, v))
    w -= quotient_in_range(ad.lr * (m * ad.inv_bc1), sqrt_in_range(fmaxf(v, 0x1p-100f)) * ad.inv_sqrt_bc2 + ad.eps);
  else
    w -= ad.lr * (m * ad.inv_bc1) / (sqrtf(v) * ad.inv_sqrt_bc2 + ad.eps);
}

// Sum over the 64 lanes of a wavefront in a fixed butterfly order; every lane
// ends with the total.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

}  // namespace gco
