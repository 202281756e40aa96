// Hidden layers in fp32 storage (widths 8 .. 128): aggregate, dense transform and epilogue.
//
// A wavefront owns a contiguous run of rows of one subgraph and takes them 16 at a time.
// Lane l = (n, h), n = l % 16, h = l / 16, works for row n of the tile and holds its
// features 16 q + 4 h + j (j = 0 .. 3): four lanes per row, 16 bytes per lane and access, a
// 64-byte segment per row and q.  That layout is at once
//   * the B operand of v_mfma_f32_16x16x4_f32 (lane (n, h): column n, contraction index h)
//     for the contraction step (q, j) over the features 16 q + 4 h + j, h = 0 .. 3, and
//   * the C/D layout of that instruction (register r of lane (n, h): row 4 h + r, column n),
// so Z^T = W^T AGG^T takes the aggregate as it stands and leaves rows in the layout they are
// stored in.  The gather has neighbouring lanes for a row (see aggregate()), and its sums change
// layout on their way through LDS.  The weight gradient contracts over the rows of the tile: its A operand (rows of
// Hprev) is read from memory in operand layout, G_T goes through wave-private LDS.
//
// Last hidden layer: its forward pass stores one bit per feature, H > 0, instead of H (unless asked for H).  Since
// dL/dZ = g_t w_out [H > 0], the backward gather sums B = A_hat^T (g_t [H > 0]) over those bits, G_T = B w_out, and with
// M = Hprev^T B:  dL/dW[a, c] = M[a, c] w_out[c],  dL/dw_out[c] = sum_a W[a, c] M[a, c]  (H = (A_hat Hprev) W where
// the bit is set).  A neighbour costs 4 to 16 bytes of bits and its g_t instead of its row: backward of the last hidden
// layer, 150 k rows of width 64, 95.5 -> 69.6 us, 700 k of width 16 with Adam 74.7 -> 62.2, forward there 33.9 -> 32.3.
//
// The aggregation walks the light stream (per row its diagonal entry, then its neighbours;
// rows with >= kHeavyMin neighbours hold only the diagonal entry and come pre-reduced): the
// tile's entries are dealt to the 16 lane groups in equal contiguous shares, whatever the
// rows look like, so a tile takes its mean and not its longest row.  A group that comes to the
// end of a row leaves the sum in LDS: in the row's place if it began the row, in the group's
// carry place if the row began in an earlier group; the row's own lanes then add its carries
// in order.  One fixed order of additions.
//
// What bounds it: at widths 8 .. 64 memory (Adam's E, m, v; the gather), so registers are kept low enough for many
// wavefronts per SIMD and there is no workgroup barrier; at width 128 the matrix cores (3 x 2 x 16 x 128 x 128
// operations per tile at 64 per cycle and SIMD).  In bytes that pass the L2s, with H stored and gathered and launch ids
// dealt round the XCDs one by one: 700 k rows of width 16, embedding backward 417 MB in 74 us, forward 144 MB in 35 (5.6
// and 4.1 TB/s); 150 k of width 64, forward 406 MB in 67 us, embedding backward 687 in 116 (5.9 to 6.1).  With contiguous
// eighths (GraphView::eighth) the latter two take 48 and 101 us.
#include "device_utils.h"
#include "gather.h"
#include "gco_internal.h"
#include "row_tiles.h"

#include <type_traits>

namespace gco {
namespace {

constexpr int kWavesPerBlock = kBlock / 64;

template <int D>
struct TK : TF<D> {
  // width 128: the weight-gradient accumulators (256 registers) are shared out over the four
  // wavefronts of the workgroup, which then advance in step
  static constexpr bool SHARED_GW = D == 128;
  static constexpr int TB = SHARED_GW ? TF<D>::NQ / kWavesPerBlock : TF<D>::NQ;  // column tiles of gW per wavefront
  static constexpr bool W_IN_LDS = D <= 64;  // width 128 reads the operands of W through the caches
};

// Rows [r0, r1) of this wavefront's run.
__device__ __forceinline__ void run_rows(const WaveRun& run, int& r0, int& r1) {
  r0 = __builtin_amdgcn_readfirstlane(run.rbeg + run.tile0 * kTile);
  r1 = __builtin_amdgcn_readfirstlane(min(run.rend, run.rbeg + run.tile1 * kTile));
}

// operand(ta, q, lane) of all tiles to LDS, wl[(ta NQ + q) 64 + lane]: all loads first, one wait.
// While they are on their way, request() starts what needs only the loads before.
template <int D, class Operand, class Request>
__device__ __forceinline__ void fill_operands(f32x4* wl, const Operand& operand, Request&& request) {
  constexpr int NQ = TK<D>::NQ;
  if constexpr (!TK<D>::W_IN_LDS) request();
  if constexpr (TK<D>::W_IN_LDS) {
    constexpr int kPer = (NQ * NQ * 64 + kBlock - 1) / kBlock;
    f32x4 v[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int idx = min(static_cast<int>(threadIdx.x) + i * kBlock, NQ * NQ * 64 - 1);
      v[i] = operand(idx / 64 / NQ, (idx / 64) % NQ, idx % 64);
    }
    loads_stay_here();
    request();
    loads_stay_here();
#pragma unroll
    for (int i = 0; i < kPer; ++i)
      if (static_cast<int>(threadIdx.x) + i * kBlock < NQ * NQ * 64) wl[threadIdx.x + i * kBlock] = v[i];
  }
}

// ---------------------------------------------------------------------------
// Forward: Y = relu((A_hat X) W^k)  [+ t = Y w_out^k]
// ---------------------------------------------------------------------------
template <int D>
constexpr size_t fwd_tile_lds() {
  return (static_cast<size_t>(TK<D>::W_IN_LDS ? TK<D>::DP * TK<D>::DP : 0) + kWavesPerBlock * TK<D>::kWaveLds +
          TK<D>::DP) *
         sizeof(float);
}

template <int D>
__global__ __launch_bounds__(kBlock, D <= 16 ? 6 : (D == 32 ? 4 : (D == 64 ? 3 : 2))) void fwd_tile_kernel(
    GraphView g, const float* __restrict__ X, const float* __restrict__ W, int w_stride, float* __restrict__ Y,
    const float* __restrict__ w_out, int wout_stride, float* __restrict__ t, uint32_t* __restrict__ mask,
    const float* __restrict__ heavy_partial) {
  constexpr int NQ = TK<D>::NQ, NM = Mask<D>::NM;
  constexpr int kTaUnroll = D <= 64 ? NQ : 1;
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4* wl = reinterpret_cast<f32x4*>(smem);
  const int tid = threadIdx.x, lane = tid % 64, n = lane % 16, h = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  const int wg = workgroup_number(g, WM_FWD);
  if (wg >= g.num_wblocks[WM_FWD]) return;
  const int k = g.wblk_k[WM_FWD][wg];
  const WaveRun run = g.wave_runs[WM_FWD][wg * kWavesPerBlock + wave];
  if (k < 0) return;
  // A operands of Z^T = W^T AGG^T: wl[(ta NQ + q) 64 + lane][j] = W[16 q + 4 h + j][16 ta + n]
  const float* Wk = W + static_cast<size_t>(k) * w_stride;
  auto w_operand = [&](int ta, int q, int l) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int f = 16 * q + 4 * (l / 16) + j, o = 16 * ta + l % 16;
      if (D >= 16 || (f < D && o < D)) v[j] = Wk[f * D + o];
    }
    return v;
  };
  // the wavefront's first tile is on its way while W is
  int r0, r1;
  run_rows(run, r0, r1);
  TileFacts<D> f, nf;
  const StreamInMemory stream{g.went, g.wrowid, g.wrowptr};
  f.request(stream, r0, r1);
  fill_operands<D>(wl, w_operand, [&]() { f.request_entries(stream); });
  float* wo = reinterpret_cast<float*>(smem + fwd_tile_lds<D>()) - TK<D>::DP;  // w_out^k
  const bool last = w_out != nullptr;
  if (last && tid < TK<D>::DP) wo[tid] = tid < D ? w_out[static_cast<size_t>(k) * wout_stride + tid] : 0.f;
  __syncthreads();
  float* sums = reinterpret_cast<float*>(smem) + (TK<D>::W_IN_LDS ? TK<D>::DP * TK<D>::DP : 0) + wave * TK<D>::kWaveLds;
  if (r0 >= r1) return;
  const PlainRows<D> rows{X};
  for (; r0 < r1; r0 += kTile) {
    const int row = r0 + n;
    nf.request(stream, r0 + kTile, r1);
    f32x4 acc[NQ];
    aggregate<D>(g, stream, rows, f, r0, r1, heavy_partial, sums, acc);
    nf.request_entries(stream);
    float part = 0.f;
    uint32_t bits[NQ];
    const int wlane = operand_lane<D>(lane);
#pragma unroll kTaUnroll
    for (int ta = 0; ta < NQ; ++ta) {
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const f32x4 w = TK<D>::W_IN_LDS ? wl[(ta * NQ + q) * 64 + wlane] : w_operand(ta, q, wlane);
#pragma unroll
        for (int j = 0; j < 4; ++j) z = mfma(w[j], acc[q][j], z);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) z[j] = fmaxf(z[j], 0.f);
      if (last) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(wo + 16 * ta + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; ++j) part = fmaf(z[j], w[j], part);
      }
      bits[ta] = 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) bits[ta] |= z[j] > 0.f ? 1u << j : 0u;
      if (row < r1 && Y != nullptr) store4<D>(Y, row, ta, h, z);
    }
    if (last) {
      part = add_over_h(part);
      uint32_t m[NM];
      row_mask<D>(h, bits, m);
      if (h == 0 && row < r1) {
        t[row] = part;
        uint32_t* to = mask + static_cast<size_t>(row) * NM;
        if constexpr (NM == 1) *to = m[0];
        else if constexpr (NM == 2) *reinterpret_cast<uint2*>(to) = make_uint2(m[0], m[1]);
        else *reinterpret_cast<uint4*>(to) = make_uint4(m[0], m[1], m[2], m[3]);
      }
    }
    f = nf;
  }
}

// ---------------------------------------------------------------------------
// Backward of a hidden layer (see BwdArgs)
// ---------------------------------------------------------------------------
template <int D>
constexpr size_t bwd_tile_lds() {
  constexpr size_t w = TK<D>::W_IN_LDS ? static_cast<size_t>(TK<D>::DP) * TK<D>::DP : 0;
  constexpr size_t gt = static_cast<size_t>(kWavesPerBlock) * TK<D>::kWaveLds;
  constexpr size_t reduce = TK<D>::SHARED_GW ? 0 : 2 * static_cast<size_t>(TK<D>::DP) * TK<D>::DP;
  return (w + (gt > reduce ? gt : reduce) + kWavesPerBlock * TK<D>::DP) * sizeof(float);
}

template <int D, bool LAST, bool TO_EMBED>
__global__ __launch_bounds__(kBlock, D <= 16 ? 4 : (D == 32 ? 3 : 2)) void bwd_tile_kernel(GraphView g, BwdArgs a) {
  using T = TK<D>;
  constexpr int NQ = T::NQ, DP = T::DP, PT = T::PT, TB = T::TB;
  constexpr WaveMap WM = TO_EMBED ? WM_EMBED : WM_BWD;
  using Rows = std::conditional_t<LAST, MaskRows<D>, PlainRows<D>>;
  constexpr int kTaUnroll = D <= 64 ? NQ : 1;
  // when the epilogue's rows are requested: as early as the registers allow
  // (ROLLING: each 16 features' worth during the products of the 16 before)
  enum { BEFORE_GATHER, AFTER_GATHER, ROLLING };
  constexpr int kState = D <= 16 || (D == 32 && !(LAST && TO_EMBED)) ? BEFORE_GATHER
                         : D == 32 || (D == 64 && !TO_EMBED)        ? AFTER_GATHER
                                                                    : ROLLING;
  constexpr int NS = kState == ROLLING ? 1 : NQ;  // groups of features held
  extern __shared__ __align__(16) unsigned char smem[];
  f32x4* wl = reinterpret_cast<f32x4*>(smem);
  float* gt_all = reinterpret_cast<float*>(smem) + (T::W_IN_LDS ? DP * DP : 0);
  float* last = reinterpret_cast<float*>(smem + bwd_tile_lds<D>()) - kWavesPerBlock * DP;
  const int wg = workgroup_number(g, WM);
  if (wg >= g.num_wblocks[WM]) return;
  const int k = g.wblk_k[WM][wg];
  if (k < 0) return;
  const AdamStep ad = a.adam.for_part(k);
  const int tid = threadIdx.x, lane = tid % 64, n = lane % 16, h = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  float* gt = gt_all + wave * T::kWaveLds;  // row sums and carries, then the G_T tile
  const float* Hprev = static_cast<const float*>(a.Hprev);  // of the first layer: E itself, which the epilogue writes
  const float* __restrict__ Wk = a.W + static_cast<size_t>(k) * a.w_stride;
  // Rows of this wavefront, kStep apart; with shared accumulators the workgroup's wavefronts
  // take turns and all of them go through the same number of tiles.
  const WaveRun* runs = g.wave_runs[WM] + wg * kWavesPerBlock;
  int r0, r1;
  constexpr int kStep = T::SHARED_GW ? kWavesPerBlock * kTile : kTile;
  if (T::SHARED_GW) {
    WaveRun all = runs[0];
    all.tile1 = runs[kWavesPerBlock - 1].tile1;
    run_rows(all, r0, r1);
    r0 += wave * kTile;
  } else {
    run_rows(runs[wave], r0, r1);
  }
  const int first = T::SHARED_GW ? r0 - wave * kTile : r0;  // of the workgroup, or of the wavefront
  TileFacts<D> f, nf;
  const StreamInMemory stream{g.went, g.wrowid, g.wrowptr};
  f.request(stream, r0, r1);
  // A operands of G_H^T = W G_T^T: [(ta NQ + q) 64 + lane][j] = W[16 ta + n][16 q + 4 h + j]
  fill_operands<D>(wl, [&](int ta, int q, int l) {
    const int o = 16 * ta + l % 16;
    return D >= 16 || o < D ? load4<D>(Wk, o, q, l / 16) : f32x4{0.f, 0.f, 0.f, 0.f};
  }, [&]() { f.request_entries(stream); });
  __syncthreads();
  // tiny subgraphs: all rows are the first wavefront's, and its sums are the workgroup's (8000 subgraphs of 3
  // rows of width 8: 32.7 -> 24.6 us, embeddings 29.4 -> 24.0)
  const bool alone = !T::SHARED_GW && runs[0].tile1 == runs[kWavesPerBlock - 1].tile1;
  if (alone && wave > 0) return;
  Rows rows;
  const float* wk = LAST ? a.w_out + static_cast<size_t>(k) * a.wout_stride : nullptr;
  f32x4 wo[LAST && D <= 64 ? NQ : 1];  // w_out, this lane's features
  if constexpr (LAST) {
    rows.mask = a.mask;
    rows.g_t = a.g_t;
    if (D <= 64) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) wo[D <= 64 ? q : 0] = load4<D>(wk, 0, q, h);
    } else {  // 32 registers less: read from LDS when used; the place receives the gradient of w_out at the end
      if (tid < D) last[tid] = wk[tid];
      __syncthreads();
    }
  } else {
    rows.X = static_cast<const float*>(a.GZ_in);
  }
  f32x4 gw[NQ][TB];
#pragma unroll
  for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) gw[ta][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
  // what the epilogue needs of the row: Adam's E, m, v, or the row of Hprev for its mask
  const bool adam = TO_EMBED && a.mode == EMBED_ADAM;
  f32x4 s_e[NS], s_m[TO_EMBED ? NS : 1], s_v[TO_EMBED ? NS : 1];
  auto request_state = [&](int row, int ta0) {  // groups ta0 .. ta0 + NS - 1
    if (!TO_EMBED || adam) {
      const int rs = min(row, r1 - 1);
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        s_e[i] = load4<D>(TO_EMBED ? a.E : Hprev, rs, ta0 + i, h);
        if (TO_EMBED) {
          s_m[TO_EMBED ? i : 0] = load4<D>(a.mE, rs, ta0 + i, h);
          s_v[TO_EMBED ? i : 0] = load4<D>(a.vE, rs, ta0 + i, h);
        }
      }
    }
  };
  for (int base = first; base < r1; base += kStep, r0 += kStep) {
    const int row = r0 + n;
    const bool valid = row < r1;
    nf.request(stream, r0 + kStep, r1);
    // rows of Hprev as the A operand of the weight gradient (contraction index h of step s:
    // row 4 s + h), requested ahead of the gather
    float av[T::SHARED_GW ? 1 : 4][NQ];
    if (!T::SHARED_GW) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int ta = 0; ta < NQ; ++ta) {
          const int hr = r0 + 4 * s + h;
          av[T::SHARED_GW ? 0 : s][ta] =
              hr < r1 && (D >= 16 || n < D) ? Hprev[static_cast<size_t>(hr) * D + 16 * ta + n] : 0.f;
        }
    }
    if (kState == BEFORE_GATHER) request_state(row, 0);
    f32x4 acc[NQ];
    aggregate<D>(g, stream, rows, f, r0, r1, a.heavy_partial, gt, acc);
    nf.request_entries(stream);
    if (kState != BEFORE_GATHER) request_state(row, 0);
    // gW[a, c] += sum over the tile's rows of Hprev[row, a] G_T[row, c]
#pragma unroll
    for (int q = 0; q < NQ; ++q) *reinterpret_cast<f32x4*>(gt + n * PT + 16 * q + 4 * h) = acc[q];
    if (T::SHARED_GW) {
      __syncthreads();
#pragma unroll 1
      for (int w = 0; w < kWavesPerBlock; ++w)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int hr = base + w * kTile + 4 * s + h;
          float hv[NQ], bv[TB];
#pragma unroll
          for (int ta = 0; ta < NQ; ++ta)
            hv[ta] = hr < r1 ? Hprev[static_cast<size_t>(hr) * D + 16 * ta + n] : 0.f;
#pragma unroll
          for (int tb = 0; tb < TB; ++tb)
            bv[tb] = gt_all[w * T::kWaveLds + (4 * s + h) * PT + 16 * (wave * TB + tb) + n];
#pragma unroll
          for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
            for (int tb = 0; tb < TB; ++tb) gw[ta][tb] = mfma(hv[ta], bv[tb], gw[ta][tb]);
        }
      __syncthreads();
    } else {
      wave_lds_handoff();
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        float bv[TB];
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) bv[tb] = gt[(4 * s + h) * PT + 16 * tb + n];
#pragma unroll
        for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) gw[ta][tb] = mfma(av[T::SHARED_GW ? 0 : s][ta], bv[tb], gw[ta][tb]);
      }
      wave_lds_handoff();
    }
    // G_Hprev^T = W G_T^T and the epilogue
    if (!(TO_EMBED && a.mode == EMBED_SKIP)) {
      const int wlane = operand_lane<D>(lane);
      if constexpr (LAST) {  // until here the sums were without w_out
#pragma unroll
        for (int q = 0; q < NQ; ++q)
          acc[q] *= D <= 64 ? wo[D <= 64 ? q : 0] : *reinterpret_cast<const f32x4*>(last + 16 * q + 4 * h);
      }
#pragma unroll kTaUnroll
      for (int ta = 0; ta < NQ; ++ta) {
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const f32x4 w = T::W_IN_LDS ? wl[(ta * NQ + q) * 64 + wlane] : load4<D>(Wk, 16 * ta + n, q, h);
#pragma unroll
          for (int j = 0; j < 4; ++j) z = mfma(w[j], acc[q][j], z);
        }
        const f32x4 hold_e = s_e[kState == ROLLING ? 0 : ta];
        f32x4 m = s_m[TO_EMBED && kState != ROLLING ? ta : 0], v = s_v[TO_EMBED && kState != ROLLING ? ta : 0];
        if (kState == ROLLING && ta + 1 < NQ) request_state(row, ta + 1);
        if (valid) {
          if (TO_EMBED) {
            if (!adam) {
              store4<D>(a.gE, row, ta, h, z);
            } else {
              f32x4 e = hold_e;
              adam_rows(ad, z, e, m, v);
              store4<D>(a.mE, row, ta, h, m);
              store4<D>(a.vE, row, ta, h, v);
              store4<D>(a.E, row, ta, h, e);
            }
          } else {
#pragma unroll
            for (int x = 0; x < 4; ++x) z[x] = hold_e[x] > 0.f ? z[x] : 0.f;
            store4<D>(static_cast<float*>(a.GZ_out), row, ta, h, z);
          }
        }
      }
    }
    f = nf;
  }

  // one partial per workgroup; LAST: M first, from which both gradients follow
  float* out = a.gW_partial + static_cast<size_t>(wg) * D * D;
  if constexpr (T::SHARED_GW) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int c = 16 * (wave * TB + tb) + n;
      const float scale = LAST ? wk[c] : 1.f;
      float column = 0.f;
#pragma unroll
      for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int at = (16 * ta + 4 * h + r) * D + c;
          if (LAST) column = fmaf(Wk[at], gw[ta][tb][r], column);
          out[at] = LAST ? gw[ta][tb][r] * scale : gw[ta][tb][r];
        }
      if (LAST) {
        column = add_over_h(column);
        if (h == 0) a.gwout_partial[static_cast<size_t>(wg) * D + c] = column;
      }
    }
  } else if (alone) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int c = 16 * tb + n;
      const bool in = D >= 16 || n < D;
      const float scale = LAST && in ? wk[c] : 1.f;
      float column = 0.f;
#pragma unroll
      for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (D >= 16 || (4 * h + r < D && in)) {
            const int at = (16 * ta + 4 * h + r) * D + c;
            if (LAST) column = fmaf(Wk[at], gw[ta][tb][r], column);
            out[at] = LAST ? gw[ta][tb][r] * scale : gw[ta][tb][r];
          }
      if (LAST) {
        column = add_over_h(column);
        if (h == 0 && in) a.gwout_partial[static_cast<size_t>(wg) * D + c] = column;
      }
    }
  } else {
    // (wave 0 + wave 2) + (wave 1 + wave 3)
    float* buf = gt_all;
    constexpr int kPer = (D * D + kBlock - 1) / kBlock;
    static_assert(kBlock % D == 0 || D > kBlock, "a thread's weights are of one column");
    float w[LAST ? kPer : 1], scale = 1.f;
    if constexpr (LAST) {
#pragma unroll
      for (int i = 0; i < kPer; ++i) w[i] = Wk[min(tid + i * kBlock, D * D - 1)];
      scale = wk[tid % D];
      loads_stay_here();
    }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
      if (wave / 2 == pass) {
        float* b = buf + (wave % 2) * DP * DP;
#pragma unroll
        for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
          for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float* p = b + (16 * ta + 4 * h + r) * DP + 16 * tb + n;
              *p = pass == 0 ? gw[ta][tb][r] : *p + gw[ta][tb][r];
            }
      }
      __syncthreads();
    }
    float column = 0.f;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int idx = tid + i * kBlock;
      if (idx < D * D) {
        const int p = (idx / D) * DP + idx % D;
        const float m = buf[p] + buf[DP * DP + p];
        if (LAST) column = fmaf(w[LAST ? i : 0], m, column);
        out[idx] = LAST ? m * scale : m;
      }
    }
    if constexpr (LAST) {
      column = column_sum<D>(column);
      if (lane < D) last[wave * DP + lane] = column;
      __syncthreads();
      if (tid < D) {
        float s = 0.f;
#pragma unroll
        for (int v = 0; v < kWavesPerBlock; ++v) s += last[v * DP + tid];
        a.gwout_partial[static_cast<size_t>(wg) * D + tid] = s;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// X = A_hat E, rows in fp32 (see launch_propagate).  The runs of the forward launch, in tiles of RT rows.
// ---------------------------------------------------------------------------
template <typename T, int D, int RT>
__global__ __launch_bounds__(kBlock) void propagate_kernel(GraphView g, const T* __restrict__ E, float* __restrict__ X,
                                                           const float* __restrict__ heavy_partial) {
  __shared__ __align__(16) float all[kWavesPerBlock * TK<D>::kWaveLds];
  const int wg = workgroup_number(g, WM_FWD);
  if (wg >= g.num_wblocks[WM_FWD] || g.wblk_k[WM_FWD][wg] < 0) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), n = threadIdx.x % 16, h = threadIdx.x % 64 / 16;
  const WaveRun run = g.wave_runs[WM_FWD][wg * kWavesPerBlock + wave];
  int r0 = __builtin_amdgcn_readfirstlane(run.rbeg + run.tile0 * RT);
  const int r1 = __builtin_amdgcn_readfirstlane(min(run.rend, run.rbeg + run.tile1 * RT));
  if (r0 >= r1) return;
  StreamWithValues stream;
  stream.went = g.went;
  stream.wrowid = g.wrowid;
  stream.wrowptr = g.wrowptr;
  stream.wval = g.wval;
  const PlainRows<D, T> rows{E};
  TileFacts<D> f, nf;
  f.request(stream, r0, r1);
  f.request_entries(stream);
  for (; r0 < r1; r0 += kTile) {
    nf.request(stream, r0 + kTile, r1);
    f32x4 acc[TK<D>::NQ];
    aggregate<D>(g, stream, rows, f, r0, r1, heavy_partial, all + wave * TK<D>::kWaveLds, acc);
    nf.request_entries(stream);
#pragma unroll
    for (int q = 0; q < TK<D>::NQ; ++q)
      if (r0 + n < r1) store4<D>(X, r0 + n, q, h, acc[q]);
    f = nf;
  }
}

template <typename T, int D, int RT>
void propagate_t(const Launch& ln, const GraphView& g, const void* E, float* X, float* heavy_partial) {
  const T* rows = static_cast<const T*>(E);
  if (g.num_chunks > 0) {
    ln.begin(KK_HEAVY);
    heavy_wide_kernel<D, PlainSrc<T, D>><<<g.num_chunks, kBlock, 0, ln.st>>>(g, PlainSrc<T, D>{rows, g.sb}, heavy_partial);
    ln.end(KK_HEAVY);
  }
  ln.begin(KK_FWD_HIDDEN);
  propagate_kernel<T, D, RT><<<launch_ids(g, WM_FWD), kBlock, 0, ln.st>>>(g, rows, X, heavy_partial);
  ln.end(KK_FWD_HIDDEN);
}

template <typename K>
void allow_lds(K kernel, size_t bytes) {
  if (bytes > 48 * 1024)
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(bytes));
}

template <int D>
void pre_reduce_t(const Launch& ln, const GraphView& g, const float* X, float* heavy_partial) {
  if (g.num_chunks == 0) return;
  ln.begin(KK_HEAVY);
  heavy_wide_kernel<D, PlainSrc<float, D>>
      <<<g.num_chunks, kBlock, 0, ln.st>>>(g, PlainSrc<float, D>{X, g.sb}, heavy_partial);
  ln.end(KK_HEAVY);
}

template <int D>
void fwd_t(const Launch& ln, const GraphView& g, const float* X, const float* W, int w_stride, float* Y,
           const float* w_out, int wout_stride, float* t, uint32_t* mask, float* heavy_partial, bool partial_ready) {
  if (!partial_ready) pre_reduce_t<D>(ln, g, X, heavy_partial);
  allow_lds(fwd_tile_kernel<D>, fwd_tile_lds<D>());
  ln.begin(KK_FWD_HIDDEN);
  fwd_tile_kernel<D><<<launch_ids(g, WM_FWD), kBlock, fwd_tile_lds<D>(), ln.st>>>(
      g, X, W, w_stride, Y, w_out, wout_stride, t, mask, heavy_partial);
  ln.end(KK_FWD_HIDDEN);
}

template <int D, bool LAST, bool TO_EMBED>
void bwd_launch(const Launch& ln, const GraphView& gt, const BwdArgs& a) {
  allow_lds(bwd_tile_kernel<D, LAST, TO_EMBED>, bwd_tile_lds<D>());
  bwd_tile_kernel<D, LAST, TO_EMBED>
      <<<launch_ids(gt, TO_EMBED ? WM_EMBED : WM_BWD), kBlock, bwd_tile_lds<D>(), ln.st>>>(gt, a);
}

template <int D>
void bwd_t(const Launch& ln, bool last, bool to_embed, const GraphView& gt, const BwdArgs& a) {
  if (gt.num_chunks > 0) {
    ln.begin(KK_HEAVY);
    if (last) {
      MaskSrc<D> src{a.mask, gt.sb, a.g_t};
      heavy_wide_kernel<D, MaskSrc<D>><<<gt.num_chunks, kBlock, 0, ln.st>>>(gt, src, a.heavy_partial);
    } else {
      PlainSrc<float, D> src{static_cast<const float*>(a.GZ_in), gt.sb};
      heavy_wide_kernel<D, PlainSrc<float, D>><<<gt.num_chunks, kBlock, 0, ln.st>>>(gt, src, a.heavy_partial);
    }
    ln.end(KK_HEAVY);
  }
  const int kind = to_embed ? KK_BWD_EMBED : KK_BWD_HIDDEN;
  ln.begin(kind);
  if (last && to_embed) bwd_launch<D, true, true>(ln, gt, a);
  else if (last) bwd_launch<D, true, false>(ln, gt, a);
  else if (to_embed) bwd_launch<D, false, true>(ln, gt, a);
  else bwd_launch<D, false, false>(ln, gt, a);
  ln.end(kind);
}

}  // namespace

#define GCO_BY_WIDTH(D, ...)                              \
  switch (D) {                                            \
    case 8: { constexpr int DD = 8; __VA_ARGS__; } break;     \
    case 16: { constexpr int DD = 16; __VA_ARGS__; } break;   \
    case 32: { constexpr int DD = 32; __VA_ARGS__; } break;   \
    case 64: { constexpr int DD = 64; __VA_ARGS__; } break;   \
    case 128: { constexpr int DD = 128; __VA_ARGS__; } break; \
    default: break;                                       \
  }

void launch_fwd_hidden_f32(const Launch& ln, int D, const GraphView& g, const void* X, const float* W,
                           int w_stride, void* Y, const float* w_out, int wout_stride, float* t,
                           uint32_t* mask, float* heavy_partial, bool partial_ready) {
  GCO_BY_WIDTH(D, (fwd_t<DD>(ln, g, static_cast<const float*>(X), W, w_stride, static_cast<float*>(Y), w_out,
                             wout_stride, t, mask, heavy_partial, partial_ready)))
}

void launch_bwd_hidden_f32(const Launch& ln, int D, bool last, bool to_embed, const GraphView& gt,
                           const BwdArgs& a) {
  GCO_BY_WIDTH(D, (bwd_t<DD>(ln, last, to_embed, gt, a)))
}

void launch_pre_reduce_f32(const Launch& ln, int D, const GraphView& g, const void* X, float* partial) {
  GCO_BY_WIDTH(D, (pre_reduce_t<DD>(ln, g, static_cast<const float*>(X), partial)))
}

void launch_propagate(const Launch& ln, int storage, int D, const GraphView& g, const void* E, float* X,
                      float* heavy_partial) {
  if (storage == GCO_STORAGE_BF16) {
    if (D == 64) propagate_t<bf16_t, 64, kWaveRows>(ln, g, E, X, heavy_partial);
    else if (D == 128) propagate_t<bf16_t, 128, kWaveRows>(ln, g, E, X, heavy_partial);
  } else {
    GCO_BY_WIDTH(D, (propagate_t<float, DD, kTileRowsF32>(ln, g, E, X, heavy_partial)))
  }
}

}  // namespace gco
