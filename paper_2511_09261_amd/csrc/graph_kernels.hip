// Integer kernels: graph checks and preprocessing at upload, cross-edge export,
// binarisation and greedy repair.  Everything here is exact.
#include "device_utils.h"
#include "graph_kernels.h"

#include <algorithm>
#include <type_traits>

namespace gco {
namespace {

// ---------------------------------------------------------------------------
// Exclusive prefix sum over int64 (three-phase, recursive on the block totals)
// ---------------------------------------------------------------------------
constexpr int kScanItems = 4;
constexpr int kScanTile = kBlock * kScanItems;

__global__ __launch_bounds__(kBlock) void scan_tiles_kernel(const int64_t* __restrict__ in,
                                                            int64_t* __restrict__ out, int64_t n,
                                                            int64_t* __restrict__ tile_sums) {
  __shared__ int64_t sh[kBlock];
  const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x * kScanItems;
  int64_t v[kScanItems];
  int64_t sum = 0;
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    v[q] = (base + q < n) ? in[base + q] : 0;
    sum += v[q];
  }
  sh[threadIdx.x] = sum;
  __syncthreads();
  for (int off = 1; off < kBlock; off <<= 1) {
    const int64_t add = threadIdx.x >= off ? sh[threadIdx.x - off] : 0;
    __syncthreads();
    sh[threadIdx.x] += add;
    __syncthreads();
  }
  int64_t run = sh[threadIdx.x] - sum;  // exclusive prefix of this thread within the tile
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    if (base + q < n) out[base + q] = run;
    run += v[q];
  }
  if (threadIdx.x == kBlock - 1) tile_sums[blockIdx.x] = sh[kBlock - 1];
}

__global__ __launch_bounds__(kBlock) void scan_add_kernel(int64_t* __restrict__ out, int64_t n,
                                                          const int64_t* __restrict__ tile_offsets) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kScanTile + threadIdx.x;
  const int64_t off = tile_offsets[blockIdx.x];
#pragma unroll
  for (int q = 0; q < kScanItems; ++q) {
    const int64_t idx = i + static_cast<int64_t>(q) * kBlock;
    if (idx < n) out[idx] += off;
  }
}

}  // namespace

size_t scan_temp_elems(int64_t n) {
  size_t total = 0;
  while (n > 1) {
    n = (n + kScanTile - 1) / kScanTile;
    total += static_cast<size_t>(n) * 2;
    if (n == 1) break;
  }
  return total + 2;
}

// out[i] = sum_{j < i} in[i] for i in [0, n]; out has n + 1 entries (out[n] = total).
// `in` must have n + 1 readable entries with in[n] ignored (treated as 0 by
// passing n + 1 items whose last is overwritten by the caller with 0).
void exclusive_scan_i64(hipStream_t st, const int64_t* in, int64_t* out, int64_t count,
                        int64_t* temp) {
  if (count <= 0) return;
  const int64_t tiles = (count + kScanTile - 1) / kScanTile;
  int64_t* sums = temp;
  int64_t* sums_scanned = temp + tiles;
  scan_tiles_kernel<<<static_cast<unsigned>(tiles), kBlock, 0, st>>>(in, out, count, sums);
  if (tiles > 1) {
    exclusive_scan_i64(st, sums, sums_scanned, tiles, temp + 2 * tiles);
    scan_add_kernel<<<static_cast<unsigned>(tiles), kBlock, 0, st>>>(out, count, sums_scanned);
  }
}

namespace {

// ---------------------------------------------------------------------------
// Upload: checks
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t row_of_entry(const int64_t* __restrict__ rowptr, int64_t n,
                                                int64_t e) {
  int64_t lo = 0, hi = n;  // last i with rowptr[i] <= e
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (rowptr[mid] <= e) lo = mid; else hi = mid;
  }
  return lo;
}

// err[0] receives the largest code seen: 1 column out of range, 2 self loop,
// 3 columns not strictly ascending, 4 missing reverse entry.
__global__ __launch_bounds__(kBlock) void check_graph_kernel(int64_t n, const int64_t* __restrict__ rowptr,
                                                             const int32_t* __restrict__ col,
                                                             int64_t nnz, int* __restrict__ err) {
  const int64_t e = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (e >= nnz) return;
  const int64_t i = row_of_entry(rowptr, n, e);
  const int64_t j = col[e];
  int code = 0;
  if (j < 0 || j >= n) {
    code = 1;
  } else if (j == i) {
    code = 2;
  } else if (e > rowptr[i] && col[e - 1] >= j) {
    code = 3;
  } else {
    int64_t lo = rowptr[j], hi = rowptr[j + 1];  // find i in row j
    bool found = false;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      const int32_t cv = col[mid];
      if (cv == i) { found = true; break; }
      if (cv < i) lo = mid + 1; else hi = mid;
    }
    if (!found) code = 4;
  }
  if (code) atomicMax(err, code);
}

// ---------------------------------------------------------------------------
// Upload: local CSR in subgraph-contiguous order
// ---------------------------------------------------------------------------
// One wavefront per new row r (original node perm[r]).
__global__ __launch_bounds__(kBlock) void local_count_kernel(int n, const int64_t* __restrict__ rowptr,
                                                             const int32_t* __restrict__ col,
                                                             const int32_t* __restrict__ part,
                                                             const int32_t* __restrict__ perm,
                                                             int64_t* __restrict__ count) {
  const int r = blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
  if (r >= n) return;
  const int lane = threadIdx.x % 64;
  const int i = perm[r];
  const int pk = part[i];
  int c = 0;
  for (int64_t e = rowptr[i] + lane; e < rowptr[i + 1]; e += 64) c += (part[col[e]] == pk) ? 1 : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if (lane == 0) count[r] = c;
}

__global__ __launch_bounds__(kBlock) void local_fill_kernel(int n, const int64_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ col,
                                                            const int32_t* __restrict__ part,
                                                            const int32_t* __restrict__ perm,
                                                            const int32_t* __restrict__ inv,
                                                            const int64_t* __restrict__ lptr64,
                                                            int32_t* __restrict__ lrowptr,
                                                            int32_t* __restrict__ lcol) {
  const int r = blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
  if (r > n) return;
  const int lane = threadIdx.x % 64;
  if (r == n) {
    if (lane == 0) lrowptr[n] = static_cast<int32_t>(lptr64[n]);
    return;
  }
  const int i = perm[r];
  const int pk = part[i];
  int64_t outp = lptr64[r];
  if (lane == 0) lrowptr[r] = static_cast<int32_t>(outp);
  const int64_t e0 = rowptr[i], e1 = rowptr[i + 1];
  for (int64_t eb = e0; eb < e1; eb += 64) {
    const int64_t e = eb + lane;
    int j = -1;
    bool keep = false;
    if (e < e1) {
      j = col[e];
      keep = part[j] == pk;
    }
    const unsigned long long mask = __ballot(keep);
    if (keep) {
      const int before = __popcll(mask & ((1ull << lane) - 1ull));
      lcol[outp + before] = inv[j];
    }
    outp += __popcll(mask);
  }
}

// sa, sb (A_hat_ij = sa_i * sb_j), the local degree and the linear coefficient.
__global__ __launch_bounds__(kBlock) void scales_kernel(int n, const int32_t* __restrict__ lrowptr,
                                                        int norm, int problem, float beta,
                                                        float* __restrict__ sa, float* __restrict__ sb,
                                                        float* __restrict__ c_base) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= n) return;
  const int deg = lrowptr[r + 1] - lrowptr[r];
  const double dt = static_cast<double>(deg) + 1.0;
  if (norm == GCO_NORM_MEAN) {
    sa[r] = static_cast<float>(1.0 / dt);
    sb[r] = 1.f;
  } else {
    const float s = static_cast<float>(1.0 / sqrt(dt));
    sa[r] = s;
    sb[r] = s;
  }
  c_base[r] = problem == GCO_PROBLEM_MAXCUT ? -static_cast<float>(deg) : -beta;
}

// One wavefront per row i: ent[e] = {j, row_scale[i] * col_scale[j]} for its entries
// e = (i, j); with diag != nullptr also diag[i] = row_scale[i] * col_scale[i].
__global__ __launch_bounds__(kBlock) void pack_entries_kernel(int n, const int32_t* __restrict__ rowptr,
                                                              const int32_t* __restrict__ col,
                                                              const float* __restrict__ row_scale,
                                                              const float* __restrict__ col_scale,
                                                              int2* __restrict__ ent,
                                                              float* __restrict__ diag) {
  const int i = blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
  if (i >= n) return;
  const int lane = threadIdx.x % 64;
  const float ri = row_scale[i];
  if (diag != nullptr && lane == 0) diag[i] = ri * col_scale[i];
  for (int e = rowptr[i] + lane; e < rowptr[i + 1]; e += 64) {
    const int j = col[e];
    ent[e] = make_int2(j, __float_as_int(ri * col_scale[j]));
  }
}

// count[i] = number of entries of row i in the light stream: its diagonal entry, and
// its neighbours unless the row is pre-reduced
__global__ __launch_bounds__(kBlock) void light_count_kernel(int n, const int32_t* __restrict__ rowptr,
                                                             int64_t* __restrict__ count) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  const int deg = rowptr[i + 1] - rowptr[i];
  count[i] = 1 + (deg >= kHeavyMin ? 0 : deg);
}

// An fp32 value as two bf16 numbers hi + lo (hi in the upper half of the word): hi is the
// value rounded to bf16, lo the rounded remainder.
__device__ __forceinline__ int split_bf16(float w) {
  const uint32_t hi = f32_to_bf16(w);
  const uint32_t lo = f32_to_bf16(w - __uint_as_float(hi << 16));
  return static_cast<int>((hi << 16) | lo);
}

// One wavefront per row: {i, diag[i]}, then a light row's entries, to the light stream,
// the values split into bf16 pairs (split) or in fp32.  wrowid (may be null) receives the row of every entry of
// the stream, -2 for the lone entry of a pre-reduced row.
__global__ __launch_bounds__(kBlock) void light_fill_kernel(int n, const int32_t* __restrict__ rowptr,
                                                            const int2* __restrict__ ent,
                                                            const float* __restrict__ diag,
                                                            const int64_t* __restrict__ wptr64,
                                                            int32_t* __restrict__ wrowptr,
                                                            int2* __restrict__ went,
                                                            float* __restrict__ wval,
                                                            int32_t* __restrict__ wrowid,
                                                            const int32_t* __restrict__ part,
                                                            const int32_t* __restrict__ perm,
                                                            const int32_t* __restrict__ part_rows,
                                                            uint32_t* __restrict__ wpair, int split) {
  const int i = blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
  if (i > n) return;
  const int lane = threadIdx.x % 64;
  if (lane == 0) wrowptr[i] = static_cast<int32_t>(wptr64[i]);
  if (i == n) return;
  const int64_t out = wptr64[i];
  const int deg = rowptr[i + 1] - rowptr[i];
  const int first = wpair != nullptr ? part_rows[part[perm[i]]] : 0;  // row of the subgraph
  if (lane == 0) {
    if (wpair != nullptr)
      wpair[out] = static_cast<uint32_t>(i - first) | (deg >= kHeavyMin ? 0xffffu : static_cast<uint32_t>(i - first)) << 16;
    went[out] = make_int2(i, split ? split_bf16(diag[i]) : __float_as_int(diag[i]));
    wval[out] = diag[i];
    if (wrowid != nullptr) wrowid[out] = deg >= kHeavyMin ? -2 : i;
  }
  if (deg >= kHeavyMin) return;
  for (int q = lane; q < deg; q += 64) {
    const int2 en = ent[rowptr[i] + q];
    went[out + 1 + q] = make_int2(en.x, split ? split_bf16(__int_as_float(en.y)) : en.y);
    wval[out + 1 + q] = __int_as_float(en.y);
    if (wrowid != nullptr) wrowid[out + 1 + q] = i;
    if (wpair != nullptr) wpair[out + 1 + q] = static_cast<uint32_t>(en.x - first) | static_cast<uint32_t>(i - first) << 16;
  }
}

// c[r] = c_base[r] + extra_orig[perm[r]]
__global__ __launch_bounds__(kBlock) void linear_coeff_kernel(int n, const float* __restrict__ c_base,
                                                              const float* __restrict__ extra_orig,
                                                              const int32_t* __restrict__ perm,
                                                              float* __restrict__ c) {
  const int r = blockIdx.x * kBlock + threadIdx.x;
  if (r >= n) return;
  c[r] = c_base[r] + (extra_orig ? extra_orig[perm[r]] : 0.f);
}

// ---------------------------------------------------------------------------
// Row permutations between original and subgraph-contiguous order
// ---------------------------------------------------------------------------
// dst[r, :] = src[map[r], :]  (width elements of 4 bytes per row)
__global__ __launch_bounds__(kBlock) void gather_rows_kernel(int64_t total, int width,
                                                             const uint32_t* __restrict__ src,
                                                             const int32_t* __restrict__ map,
                                                             uint32_t* __restrict__ dst) {
  const int64_t idx = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= total) return;
  const int64_t r = idx / width;
  const int c = static_cast<int>(idx % width);
  dst[idx] = src[static_cast<int64_t>(map[r]) * width + c];
}

__global__ __launch_bounds__(kBlock) void gather_bytes_kernel(int n, const uint8_t* __restrict__ src,
                                                              const int32_t* __restrict__ map,
                                                              uint8_t* __restrict__ dst) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) dst[i] = src[map[i]];
}

// ---------------------------------------------------------------------------
// Cross edges
// ---------------------------------------------------------------------------
// The kernels over all entries of the full CSR take kEntryChunk consecutive entries per workgroup,
// eight per thread, whatever the rows look like: rows have five entries on average and up to
// tens of thousands, so that a wavefront per row (the form before) spent its time on rows
// shorter than itself (1.1 M rows, 6 M entries: count of the cross edges 238 -> 31 us, their list
// 241 -> 37, edge counts 282 -> 34).  What is left is the latency of a chunk's search for its rows
// and of the scattered looks at the other ends.
constexpr int kEntryChunk = 8 * kBlock;
constexpr int kRowWalk = 32;  // x kBlock rows of a chunk are walked; four times its entries

struct RowsScratch {
  alignas(16) int mark[kEntryChunk];
  int wave_top[kBlock / 64];
};

// The rows of entries e0 + 8 tid .. + 7 of the workgroup's chunk [e0, e1).  Contains barriers.
__device__ void rows_of_entries(const int64_t* __restrict__ rowptr, int n, int64_t e0, int64_t e1, RowsScratch& sh,
                                int (&row)[8]) {
  const int tid = threadIdx.x, lane = tid % 64, wave = tid / 64;
  // the last row that begins at or before e0: 64 places are looked at at once
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) / 64;
    const int64_t at = static_cast<int64_t>(lo) + static_cast<int64_t>(lane + 1) * step;
    const bool before = at < hi && rowptr[at] <= e0;
    const int passed = __popcll(__ballot(before));
    const int64_t end = static_cast<int64_t>(lo) + static_cast<int64_t>(passed + 1) * step;
    lo += passed * step;
    hi = static_cast<int>(min(end, static_cast<int64_t>(hi)));
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) sh.mark[i * kBlock + tid] = -1;
  __syncthreads();
  if (tid == 0) sh.mark[0] = lo;
  // every later row that begins inside the chunk leaves its number there (of several that begin
  // at one place the last one has entries)
  bool more = true;
  int64_t r = static_cast<int64_t>(lo) + 1 + tid;
  for (int i = 0; more && i < kRowWalk; ++i, r += kBlock) {
    const int64_t at = r < n ? rowptr[r] : e1;
    more = at < e1;
    if (more && at > e0) atomicMax(&sh.mark[at - e0], static_cast<int>(r));
  }
  if (__syncthreads_or(more)) {
    // far more rows than entries (nodes without edges): each entry looks for its row by itself
#pragma unroll 1
    for (int i = 0; i < 8; ++i) {
      const int64_t e = e0 + 8 * tid + i;
      int a = lo, b = n;
      while (b - a > 1) {
        const int mid = a + (b - a) / 2;
        if (rowptr[mid] <= e) a = mid; else b = mid;
      }
      sh.mark[8 * tid + i] = a;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) row[i] = sh.mark[8 * tid + i];
    return;
  }
  // running maximum over the chunk
  int top = -1;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    top = max(top, sh.mark[8 * tid + i]);
    row[i] = top;
  }
  int scan = top;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int other = __shfl_up(scan, off, 64);
    if (lane >= off) scan = max(scan, other);
  }
  if (lane == 63) sh.wave_top[wave] = scan;
  int before = __shfl_up(scan, 1, 64);
  if (lane == 0) before = -1;
  __syncthreads();
  for (int w = 0; w < wave; ++w) before = max(before, sh.wave_top[w]);
#pragma unroll
  for (int i = 0; i < 8; ++i) row[i] = max(row[i], before);
}

// Columns of entries e0 + 8 tid .. + 7 (-1 past e1; col starts at a 16-byte boundary).
__device__ __forceinline__ void columns_of_entries(const int32_t* __restrict__ col, int64_t e0, int64_t e1,
                                                   int (&j)[8]) {
  const int64_t e = e0 + 8 * threadIdx.x;
  if (e + 8 <= e1) {
    const int4 a = *reinterpret_cast<const int4*>(col + e), b = *reinterpret_cast<const int4*>(col + e + 4);
    j[0] = a.x; j[1] = a.y; j[2] = a.z; j[3] = a.w;
    j[4] = b.x; j[5] = b.y; j[6] = b.z; j[7] = b.w;
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) j[i] = e + i < e1 ? col[e + i] : -1;
  }
}

// Bit i: entry (row[i], j[i]) is an edge between subgraphs, seen from its smaller end (and, with x,
// both ends are selected).
__device__ __forceinline__ unsigned cross_bits(const int (&row)[8], const int (&j)[8],
                                               const int32_t* __restrict__ part, const uint8_t* __restrict__ x) {
  unsigned bits = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (j[i] > row[i] && part[row[i]] != part[j[i]] && (x == nullptr || (x[row[i]] && x[j[i]]))) bits |= 1u << i;
  return bits;
}

// count[b] = cross edges among the entries of chunk b
__global__ __launch_bounds__(kBlock) void cut_count_kernel(int n, int64_t nnz, const int64_t* __restrict__ rowptr,
                                                           const int32_t* __restrict__ col,
                                                           const int32_t* __restrict__ part,
                                                           const uint8_t* __restrict__ x,
                                                           int64_t* __restrict__ count) {
  __shared__ RowsScratch sh;
  __shared__ int sums[kBlock / 64];
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kEntryChunk, e1 = min(e0 + kEntryChunk, nnz);
  int row[8], j[8];
  columns_of_entries(col, e0, e1, j);
  rows_of_entries(rowptr, n, e0, e1, sh, row);
  int c = __popc(cross_bits(row, j, part, x));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if (threadIdx.x % 64 == 0) sums[threadIdx.x / 64] = c;
  __syncthreads();
  if (threadIdx.x == 0) count[blockIdx.x] = sums[0] + sums[1] + sums[2] + sums[3];
}

// The edges of chunk b, in the order of the entries, from place offs[b] on.
__global__ __launch_bounds__(kBlock) void cut_fill_kernel(int n, int64_t nnz, const int64_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ col,
                                                          const int32_t* __restrict__ part,
                                                          const uint8_t* __restrict__ x,
                                                          const int64_t* __restrict__ offs, int32_t* __restrict__ u,
                                                          int32_t* __restrict__ v) {
  __shared__ RowsScratch sh;
  __shared__ int sums[kBlock / 64];
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kEntryChunk, e1 = min(e0 + kEntryChunk, nnz);
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  int row[8], j[8];
  columns_of_entries(col, e0, e1, j);
  rows_of_entries(rowptr, n, e0, e1, sh, row);
  const unsigned bits = cross_bits(row, j, part, x);
  const int c = __popc(bits);
  int scan = c;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int other = __shfl_up(scan, off, 64);
    if (lane >= off) scan += other;
  }
  if (lane == 63) sums[wave] = scan;
  __syncthreads();
  int64_t at = offs[blockIdx.x] + scan - c;
  for (int w = 0; w < wave; ++w) at += sums[w];
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (bits >> i & 1u) {
      u[at] = row[i];
      v[at] = j[i];
      ++at;
    }
}

// cross[i] = 1 for both ends of every cross edge
__global__ __launch_bounds__(kBlock) void cross_mark_kernel(int n, int64_t nnz, const int64_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ col,
                                                            const int32_t* __restrict__ part,
                                                            uint8_t* __restrict__ cross) {
  __shared__ RowsScratch sh;
  const int64_t e0 = static_cast<int64_t>(blockIdx.x) * kEntryChunk, e1 = min(e0 + kEntryChunk, nnz);
  int row[8], j[8];
  columns_of_entries(col, e0, e1, j);
  rows_of_entries(rowptr, n, e0, e1, sh, row);
  // every edge is stored in both directions: marking the row of each entry marks both ends
#pragma unroll
  for (int i = 0; i < 8; ++i)
    if (j[i] >= 0 && part[row[i]] != part[j[i]]) cross[row[i]] = 1;
}

// ---------------------------------------------------------------------------
// Binarisation, greedy repair, counts
// ---------------------------------------------------------------------------
// state: 0 = not selected or removed, 1 = selected and undecided, 2 = kept
__global__ __launch_bounds__(kBlock) void round_kernel(int n, const float* __restrict__ p, float thr,
                                                       uint8_t* __restrict__ state) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) state[i] = p[i] >= thr ? 1 : 0;
}

// kLanes lanes per undecided node; the whole workgroup, afterwards, for nodes with more than
// kRepairOwn kLanes neighbours.  A node is removed once a kept neighbour
// of higher priority exists, kept once every selected neighbour of higher
// priority has been removed.  Priority: p descending, then index ascending.
// States only move 1 -> 0 or 1 -> 2 and every decision rests on final facts,
// so the fixed point does not depend on the interleaving.
// Bound by latency: column, then its state and probability.  With a wavefront per node and an
// atomic count of the undecided, the first round over 1.1 M nodes took 416 us, now 56; the mean of
// eight rounds 153 against 22.  Eight lanes suit rows of a few neighbours; where most nodes have more
// than their share of 128 and would fall to the workgroup, one after another, a node takes a wavefront
// (repair over all edges, 4 k nodes of 200 neighbours: 448 -> 281 us, 3 k of 1000: 438 -> 308; but
// 20 k of 100: 330 with eight lanes, 418 with a wavefront).
constexpr int kRepairOwn = 16;

template <int kLanes, typename PtrT>
__global__ __launch_bounds__(kBlock) void repair_round_kernel(int n, const PtrT* __restrict__ rowptr,
                                                              const int32_t* __restrict__ col,
                                                              const float* __restrict__ p,
                                                              volatile uint8_t* state,
                                                              int* __restrict__ undecided) {
  constexpr int kAtOnce = kLanes == 64 ? 4 : 2;  // entries of a lane in flight
  __shared__ int longs[kBlock / kLanes];
  __shared__ int num_longs;
  const int tid = threadIdx.x, lane = tid % 64, sub = tid % kLanes;
  const int i = blockIdx.x * (kBlock / kLanes) + tid / kLanes;
  if (tid == 0) num_longs = 0;
  __syncthreads();
  const bool open = i < n && state[i] == 1;
  PtrT e0 = 0, e1 = 0;
  float pi = 0.f;
  if (open) {
    e0 = rowptr[i];
    e1 = rowptr[i + 1];
    pi = p[i];
  }
  bool kill = false, wait = false;
  // what the entries e, e + step, ... of node `me` of probability `pm` say of it
  auto look = [&](PtrT e, PtrT end, int step, int me, float pm, auto slots) {
    constexpr int N = decltype(slots)::value;
    int j[N], sj[N];
    float pj[N];
#pragma unroll
    for (int u = 0; u < N; ++u) j[u] = e + u * step < end ? col[e + u * step] : -1;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      sj[u] = j[u] >= 0 ? state[j[u]] : 0;
      pj[u] = j[u] >= 0 ? p[j[u]] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const bool above = sj[u] != 0 && (pj[u] > pm || (pj[u] == pm && j[u] < me));
      kill |= above && sj[u] == 2;
      wait |= above && sj[u] != 2;
    }
  };
  const bool own = e1 - e0 <= kRepairOwn * kLanes;
  const PtrT end = own ? e1 : e0;
  for (PtrT e = e0 + sub; __any(e < end); e += kAtOnce * kLanes) {
    look(e, end, kLanes, i, pi, std::integral_constant<int, kAtOnce>{});
    if (kLanes == 64 && __any(kill)) break;
  }
  const unsigned long long group = kLanes == 64 ? ~0ull : ((1ull << (kLanes % 64)) - 1ull) << (lane - sub);
  const bool any_kill = (__ballot(kill) & group) != 0, any_wait = (__ballot(wait) & group) != 0;
  bool left = false;
  if (open && sub == 0) {
    if (!own) longs[atomicAdd(&num_longs, 1)] = i;
    else if (any_kill) state[i] = 0;
    else if (!any_wait) state[i] = 2;
    else left = true;
  }
  __syncthreads();
  for (int q = 0; q < num_longs; ++q) {
    const int me = longs[q];
    const PtrT b = rowptr[me], t = rowptr[me + 1];
    const float pm = p[me];
    kill = wait = false;
    for (PtrT e = b; e < t; e += 8 * kBlock) {
      look(e + tid, t, kBlock, me, pm, std::integral_constant<int, 8>{});
      if (__syncthreads_or(kill)) break;
    }
    const bool killed = __syncthreads_or(kill), waits = __syncthreads_or(wait);
    if (killed) {
      if (tid == 0) state[me] = 0;
    } else if (!waits) {
      if (tid == 0) state[me] = 2;
    } else {
      left = true;
    }
  }
  // every store writes the same value
  if (undecided != nullptr && __any(left) && lane == 0) *undecided = 1;
}

__global__ __launch_bounds__(kBlock) void state_to_x_kernel(int n, const uint8_t* __restrict__ state,
                                                            uint8_t* __restrict__ x) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i < n) x[i] = state[i] != 0 ? 1 : 0;
}

// counts[0] += |{i: x_i = 1}|, counts[1] += edges with both ends 1,
// counts[2] += edges whose ends differ (each undirected edge once, i < j).
__global__ __launch_bounds__(kBlock) void edge_counts_kernel(int n, int64_t nnz, const int64_t* __restrict__ rowptr,
                                                             const int32_t* __restrict__ col,
                                                             const uint8_t* __restrict__ x,
                                                             unsigned long long* __restrict__ counts) {
  // integer sums are combined per workgroup before the three atomics, so the totals are exact
  // and contention is low; the nodes are dealt to the workgroups in equal runs
  __shared__ RowsScratch sh;
  __shared__ unsigned int part[3][kBlock / 64];
  const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
  unsigned int sel = 0, both = 0, differ = 0;
  const int64_t run = (static_cast<int64_t>(n) + gridDim.x - 1) / gridDim.x;
  for (int64_t i = blockIdx.x * run + threadIdx.x; i < min((blockIdx.x + 1) * run, static_cast<int64_t>(n)); i += kBlock)
    sel += x[i];
  for (int64_t e0 = static_cast<int64_t>(blockIdx.x) * kEntryChunk; e0 < nnz;
       e0 += static_cast<int64_t>(gridDim.x) * kEntryChunk) {
    const int64_t e1 = min(e0 + kEntryChunk, nnz);
    int row[8], j[8];
    columns_of_entries(col, e0, e1, j);
    __syncthreads();  // the marks of the chunk before have been read
    rows_of_entries(rowptr, n, e0, e1, sh, row);
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (j[i] > row[i]) {
        const int xi = x[row[i]], xj = x[j[i]];
        both += (xi & xj);
        differ += (xi ^ xj);
      }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    sel += __shfl_xor(sel, off, 64);
    both += __shfl_xor(both, off, 64);
    differ += __shfl_xor(differ, off, 64);
  }
  if (lane == 0) {
    part[0][wave] = sel;
    part[1][wave] = both;
    part[2][wave] = differ;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    unsigned long long tot = 0;
    for (int w = 0; w < kBlock / 64; ++w) tot += part[threadIdx.x][w];
    if (tot) atomicAdd(&counts[threadIdx.x], tot);
  }
}

__global__ __launch_bounds__(kBlock) void fill_u32_kernel(uint32_t* __restrict__ dst, int64_t count,
                                                          uint32_t value) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * kBlock + threadIdx.x;
  if (i < count) dst[i] = value;
}

inline unsigned blocks_for(int64_t items, int per_block) {
  return static_cast<unsigned>((items + per_block - 1) / per_block);
}

}  // namespace

void launch_check_graph(hipStream_t st, int64_t n, const int64_t* rowptr, const int32_t* col,
                        int64_t nnz, int* err) {
  if (nnz > 0) check_graph_kernel<<<blocks_for(nnz, kBlock), kBlock, 0, st>>>(n, rowptr, col, nnz, err);
}

void launch_local_count(hipStream_t st, int n, const int64_t* rowptr, const int32_t* col,
                        const int32_t* part, const int32_t* perm, int64_t* count) {
  local_count_kernel<<<blocks_for(n, kBlock / 64), kBlock, 0, st>>>(n, rowptr, col, part, perm, count);
}

void launch_local_fill(hipStream_t st, int n, const int64_t* rowptr, const int32_t* col,
                       const int32_t* part, const int32_t* perm, const int32_t* inv,
                       const int64_t* lptr64, int32_t* lrowptr, int32_t* lcol) {
  local_fill_kernel<<<blocks_for(static_cast<int64_t>(n) + 1, kBlock / 64), kBlock, 0, st>>>(
      n, rowptr, col, part, perm, inv, lptr64, lrowptr, lcol);
}

void launch_scales(hipStream_t st, int n, const int32_t* lrowptr, int norm, int problem, float beta,
                   float* sa, float* sb, float* c_base) {
  scales_kernel<<<blocks_for(n, kBlock), kBlock, 0, st>>>(n, lrowptr, norm, problem, beta, sa, sb, c_base);
}

void launch_pack_entries(hipStream_t st, int n, const int32_t* rowptr, const int32_t* col,
                         const float* row_scale, const float* col_scale, int2* ent, float* diag) {
  pack_entries_kernel<<<blocks_for(n, kBlock / 64), kBlock, 0, st>>>(n, rowptr, col, row_scale, col_scale,
                                                                      ent, diag);
}

void launch_light_count(hipStream_t st, int n, const int32_t* rowptr, int64_t* count) {
  light_count_kernel<<<blocks_for(n, kBlock), kBlock, 0, st>>>(n, rowptr, count);
}

void launch_light_fill(hipStream_t st, int n, const int32_t* rowptr, const int2* ent, const float* diag,
                       const int64_t* wptr64, int32_t* wrowptr, int2* went, float* wval, int32_t* wrowid,
                       const int32_t* part, const int32_t* perm, const int32_t* part_rows, uint32_t* wpair, bool split) {
  light_fill_kernel<<<blocks_for(static_cast<int64_t>(n) + 1, kBlock / 64), kBlock, 0, st>>>(
      n, rowptr, ent, diag, wptr64, wrowptr, went, wval, wrowid, part, perm, part_rows, wpair, split ? 1 : 0);
}

void launch_linear_coeff(hipStream_t st, int n, const float* c_base, const float* extra_orig,
                         const int32_t* perm, float* c) {
  linear_coeff_kernel<<<blocks_for(n, kBlock), kBlock, 0, st>>>(n, c_base, extra_orig, perm, c);
}

void launch_gather_rows(hipStream_t st, int64_t rows, int width, const void* src, const int32_t* map,
                        void* dst) {
  const int64_t total = rows * width;
  if (total > 0)
    gather_rows_kernel<<<blocks_for(total, kBlock), kBlock, 0, st>>>(
        total, width, static_cast<const uint32_t*>(src), map, static_cast<uint32_t*>(dst));
}

void launch_gather_bytes(hipStream_t st, int n, const uint8_t* src, const int32_t* map, uint8_t* dst) {
  gather_bytes_kernel<<<blocks_for(n, kBlock), kBlock, 0, st>>>(n, src, map, dst);
}

int64_t entry_chunks(int64_t nnz) { return (nnz + kEntryChunk - 1) / kEntryChunk; }

void launch_cut_count(hipStream_t st, int n, int64_t nnz, const int64_t* rowptr, const int32_t* col,
                      const int32_t* part, const uint8_t* x, int64_t* count) {
  if (nnz > 0)
    cut_count_kernel<<<static_cast<unsigned>(entry_chunks(nnz)), kBlock, 0, st>>>(n, nnz, rowptr, col, part, x, count);
}

void launch_cut_fill(hipStream_t st, int n, int64_t nnz, const int64_t* rowptr, const int32_t* col,
                     const int32_t* part, const uint8_t* x, const int64_t* offs, int32_t* u, int32_t* v) {
  if (nnz > 0)
    cut_fill_kernel<<<static_cast<unsigned>(entry_chunks(nnz)), kBlock, 0, st>>>(n, nnz, rowptr, col, part, x, offs, u, v);
}

void launch_cross_mark(hipStream_t st, int n, int64_t nnz, const int64_t* rowptr, const int32_t* col,
                       const int32_t* part, uint8_t* cross) {
  if (nnz > 0)
    cross_mark_kernel<<<static_cast<unsigned>(entry_chunks(nnz)), kBlock, 0, st>>>(n, nnz, rowptr, col, part, cross);
}

void launch_round(hipStream_t st, int n, const float* p, float thr, uint8_t* state) {
  round_kernel<<<blocks_for(n, kBlock), kBlock, 0, st>>>(n, p, thr, state);
}

template <typename PtrT>
static void repair_round(hipStream_t st, int n, int64_t nnz, const PtrT* rowptr, const int32_t* col, const float* p,
                         uint8_t* state, int* undecided) {
  if (nnz < 8 * kRepairOwn * static_cast<int64_t>(n))
    repair_round_kernel<8><<<blocks_for(n, kBlock / 8), kBlock, 0, st>>>(n, rowptr, col, p, state, undecided);
  else
    repair_round_kernel<64><<<blocks_for(n, kBlock / 64), kBlock, 0, st>>>(n, rowptr, col, p, state, undecided);
}

void launch_repair_round_local(hipStream_t st, int n, int64_t nnz, const int32_t* lrowptr, const int32_t* lcol,
                               const float* p, uint8_t* state, int* undecided) {
  repair_round(st, n, nnz, lrowptr, lcol, p, state, undecided);
}

void launch_repair_round_all(hipStream_t st, int n, int64_t nnz, const int64_t* rowptr, const int32_t* col,
                             const float* p, uint8_t* state, int* undecided) {
  repair_round(st, n, nnz, rowptr, col, p, state, undecided);
}

void launch_state_to_x(hipStream_t st, int n, const uint8_t* state, uint8_t* x) {
  state_to_x_kernel<<<blocks_for(n, kBlock), kBlock, 0, st>>>(n, state, x);
}

void launch_edge_counts(hipStream_t st, int n, int64_t nnz, const int64_t* rowptr, const int32_t* col,
                        const uint8_t* x, unsigned long long* counts) {
  // four workgroups per CU: the atomics of one per chunk took longer than the counting (3 k chunks:
  // 49 us against 34); at least one, since without entries the nodes are counted all the same
  const int64_t chunks = std::min<int64_t>(1024, std::max<int64_t>(1, entry_chunks(nnz)));
  edge_counts_kernel<<<static_cast<unsigned>(chunks), kBlock, 0, st>>>(n, nnz, rowptr, col, x, counts);
}

void launch_fill_u32(hipStream_t st, void* dst, int64_t count, uint32_t value) {
  if (count > 0)
    fill_u32_kernel<<<blocks_for(count, kBlock), kBlock, 0, st>>>(static_cast<uint32_t*>(dst), count, value);
}

}  // namespace gco
