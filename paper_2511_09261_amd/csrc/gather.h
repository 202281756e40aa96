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
  __device__ __forceinline__ void load(int j, int c0, float (&v)[VEC]) const {
    Store<T>::load(X + static_cast<size_t>(j) * D + c0, v);
    const float s = sb[j];
#pragma unroll
    for (int x = 0; x < VEC; ++x) v[x] *= s;
  }
};

// Gradient of the last hidden layer's pre-activation without the factor w_out:
// v = sb[j] * g_t[j] where bit c of row j's mask (bit c % 32 of word c / 32) is set
template <int D>
struct MaskSrc {
  static constexpr int VEC = 4;
  const uint32_t* mask;
  const float* sb;
  const float* g_t;
  __device__ __forceinline__ void load(int j, int c0, float (&v)[VEC]) const {
    const uint32_t m = mask[static_cast<size_t>(j) * ((D + 31) / 32) + c0 / 32] >> (c0 % 32);
    const float s = sb[j] * g_t[j];
#pragma unroll
    for (int x = 0; x < VEC; ++x) v[x] = (m >> x) & 1u ? s : 0.f;
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

// Chunked pre-reduction of very long rows: partial[c, :] = sum_{e in chunk c} src(col[e]), by one workgroup; red is
// kBlock * VEC floats of its LDS.
template <int D, class Src>
__device__ __forceinline__ void reduce_chunk_of(const GraphView& g, Src src, float* __restrict__ partial, int ch, float* red) {
  constexpr int VEC = Src::VEC;
  constexpr int LPR = D / VEC;
  constexpr int G = kBlock / LPR;
  const int tid = threadIdx.x;
  const int grp = tid / LPR;
  const int c0 = (tid % LPR) * VEC;
  if (g.chunk_part[ch] < 0) return;  // the row's subgraph sits out
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

template <int D, class Src>
__global__ __launch_bounds__(kBlock) void heavy_wide_kernel(GraphView g, Src src, float* partial) {
  __shared__ float red[kBlock * Src::VEC];
  reduce_chunk_of<D>(g, src, partial, blockIdx.x, red);
}

}  // namespace gco
