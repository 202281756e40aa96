// Pre-reduction of the rows with very many neighbours (fp32 storage): the sources of
// gathered rows, the fixed-order row gather and the kernel over the chunks.
#pragma once

#include "device_utils.h"
#include "gco_internal.h"

namespace gco {

// ---------------------------------------------------------------------------
// Sources of gathered rows
// ---------------------------------------------------------------------------

// v = sb[j] * X[j, c0 .. c0+VEC)
template <typename T, int D>
struct PlainSrc {
  static constexpr int VEC = Store<T>::VEC;
  const T* X;
  const float* sb;
  __device__ __forceinline__ void set_part(int, int) {}
  __device__ __forceinline__ void load(int j, int c0, float (&v)[VEC]) const {
    Store<T>::load(X + static_cast<size_t>(j) * D + c0, v);
    const float s = sb[j];
#pragma unroll
    for (int x = 0; x < VEC; ++x) v[x] *= s;
  }
};

// Gradient of the last hidden layer's pre-activation, formed on the fly:
// v = sb[j] * g_t[j] * w_out[c] * [H[j, c] > 0]
template <typename T, int D>
struct LastSrc {
  static constexpr int VEC = Store<T>::VEC;
  const T* H;
  const float* sb;
  const float* g_t;
  const float* w_out;  // [Pw, D]
  int wout_stride;
  float w[VEC];
  __device__ __forceinline__ void set_part(int k, int c0) {
#pragma unroll
    for (int x = 0; x < VEC; ++x) w[x] = w_out[static_cast<size_t>(k) * wout_stride + c0 + x];
  }
  __device__ __forceinline__ void load(int j, int c0, float (&v)[VEC]) const {
    Store<T>::load(H + static_cast<size_t>(j) * D + c0, v);
    const float s = sb[j] * g_t[j];
#pragma unroll
    for (int x = 0; x < VEC; ++x) v[x] = v[x] > 0.f ? s * w[x] : 0.f;
  }
};

// acc += sum over entries e0, e0+stride, ... < e1 of src(col[e]); four rows in flight.
template <class Src>
__device__ __forceinline__ void gather_range(const Src& src, const int* __restrict__ col, int e0,
                                             int e1, int stride, int c0,
                                             float (&acc)[Src::VEC]) {
  constexpr int VEC = Src::VEC;
  int e = e0;
  for (; e + 3 * stride < e1; e += 4 * stride) {
    const int j0 = col[e], j1 = col[e + stride], j2 = col[e + 2 * stride], j3 = col[e + 3 * stride];
    float v0[VEC], v1[VEC], v2[VEC], v3[VEC];
    src.load(j0, c0, v0);
    src.load(j1, c0, v1);
    src.load(j2, c0, v2);
    src.load(j3, c0, v3);
#pragma unroll
    for (int x = 0; x < VEC; ++x) acc[x] = (((acc[x] + v0[x]) + v1[x]) + v2[x]) + v3[x];
  }
  for (; e < e1; e += stride) {
    float v0[VEC];
    src.load(col[e], c0, v0);
#pragma unroll
    for (int x = 0; x < VEC; ++x) acc[x] += v0[x];
  }
}

// Chunked pre-reduction of very long rows: partial[c, :] = sum_{e in chunk c} src(col[e]).
template <int D, class Src>
__global__ __launch_bounds__(kBlock) void heavy_wide_kernel(GraphView g, Src src, float* partial) {
  constexpr int VEC = Src::VEC;
  constexpr int LPR = D / VEC;
  constexpr int G = kBlock / LPR;
  __shared__ float red[kBlock * VEC];
  const int ch = blockIdx.x;
  const int tid = threadIdx.x;
  const int grp = tid / LPR;
  const int c0 = (tid % LPR) * VEC;
  if (g.chunk_part[ch] < 0) return;  // the row's subgraph sits out
  src.set_part(g.chunk_part[ch], c0);
  float acc[VEC];
#pragma unroll
  for (int x = 0; x < VEC; ++x) acc[x] = 0.f;
  gather_range(src, g.col, g.chunk_begin[ch] + grp, g.chunk_end[ch], G, c0, acc);
#pragma unroll
  for (int x = 0; x < VEC; ++x) red[grp * D + c0 + x] = acc[x];
  __syncthreads();
  if (tid < D) {
    float s = 0.f;
    for (int gq = 0; gq < G; ++gq) s += red[gq * D + tid];
    partial[static_cast<size_t>(ch) * D + tid] = s;
  }
}

}  // namespace gco
