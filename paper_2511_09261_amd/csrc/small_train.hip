// Training epochs of small subgraphs in ONE launch: a workgroup per subgraph runs whole epochs
// (forward, loss, backward, Adam) one after another, up to kLossSets of them per launch.
//
// Subgraphs are independent (Sec. 3.3), so with weights of their own nothing crosses a
// workgroup: the phases of an epoch are separated by workgroup barriers (a fraction of a
// microsecond) instead of launches (5 us and more each, four to eight per epoch).  The
// subgraph's light stream, its row offsets, its weight matrices and every width-1 vector stay in
// LDS for all epochs; features, gradients and the optimizer's state are read from and written to
// memory, where they stay in the caches of the one compute unit that uses them.
//
// The wide phases use the tile code of row_tiles.h (16 rows per wavefront at a time, tiles dealt
// to the wavefronts in turn), the width-1 phases a segmented scan over the stream in LDS
// (64 entries per step, whole rows per wavefront).  bf16 storage rounds where the launches of
// its own do (stored features and gradients, the operands of the dense products) and multiplies
// the rounded values on the fp32 matrix instructions, which is exact per product.
//
// Best-by-loss snapshots are taken inside the epoch, between the loss and the update, so that tracking
// them costs no second forward pass and no launch.
//
// What bounds it: the chain of dependent phases -- per epoch about ten barriers, and per tile the
// latency of its gather and of its products.
#include "device_utils.h"
#include "gco_internal.h"
#include "row_tiles.h"
#include "segmented_scan.h"

#include <algorithm>
#include <type_traits>

namespace gco {
namespace {

// zero entries after the stream in LDS: a tile dealt row by row reads a longest row (below
// kHeavyMin neighbours and the diagonal) and two batches past its last row's beginning
constexpr int kSmallPad = kHeavyMin + 16;

template <int D>
struct SK : TF<D> {
  static constexpr int NW = D <= 32 ? 16 : 8;  // wavefronts of the workgroup
  static constexpr int NT = 64 * NW;
  static constexpr int WP = TF<D>::DP + 4;  // pitch of a weight matrix in LDS (floats)
  static constexpr int kW = TF<D>::DP * WP;
};

// The workgroup's LDS, in floats from its start.
template <int D>
struct Carve {
  size_t w[2], wo, sums, gwo, c, t, p, rp, ent, valt, red, end;
  __host__ __device__ Carve(int L, int rows, int entries, bool mean) {
    const size_t r = (static_cast<size_t>(rows) + 7) / 4 * 4;
    const size_t e = (static_cast<size_t>(entries) + kSmallPad + 3) / 4 * 4;
    size_t at = 0;
    auto take = [&](size_t floats) {
      const size_t x = at;
      at += (floats + 3) / 4 * 4;
      return x;
    };
    w[0] = take(SK<D>::kW);
    w[1] = L == 3 ? take(SK<D>::kW) : 0;
    wo = take(SK<D>::DP);
    sums = take(static_cast<size_t>(SK<D>::NW) * SK<D>::kWaveLds);
    gwo = take(static_cast<size_t>(SK<D>::NW) * SK<D>::DP);
    c = take(r);
    t = take(r);
    p = take(r);
    rp = take(r);
    ent = take(2 * e);
    valt = mean ? take(e) : 0;
    red = take(2 * SK<D>::NW + 4);  // the wavefronts' shares of the loss, the lowest loss, whether this one is lower
    end = at;
  }
};

// The light stream of the subgraph in LDS: rows and columns relative to its first row, 16 bits
// each, and the entry's value (of A_hat, or of its transpose where that differs).
struct StreamInLds {
  const uint2* ent;
  const float* valt;  // nullptr: the values of ent
  const int* rp;
  static constexpr bool kPreReduced = false;
  static __device__ __forceinline__ bool by_row(int longest, int share) { return longest <= 3 * (share + 1); }
  __device__ __forceinline__ int begin_of(int row) const { return rp[row]; }
  __device__ __forceinline__ Entry at(int e) const {
    const uint2 x = ent[e];
    return Entry{static_cast<int>(x.x & 0xffffu), static_cast<int>(x.x >> 16),
                 valt != nullptr ? valt[e] : __uint_as_float(x.y)};
  }
};

// finish(row, sum of the row's terms) for the rows whose entries fill [e0, e1) of the stream, by one
// wavefront; term(entry) is an entry's contribution.
template <class Term, class Finish>
__device__ __forceinline__ void scan_rows(const StreamInLds& s, int e0, int e1, Term&& term, Finish&& finish) {
  const int lane = threadIdx.x % 64;
  int carry_row = -1;
  float carry = 0.f;
  for (int b = e0; b < e1; b += 64) {
    const bool ok = b + lane < e1;
    const Entry en = s.at(ok ? b + lane : e0);
    const int row = ok ? en.row : -1;
    float v = ok ? term(en) : 0.f;
    const int after = b + 64 < e1 ? s.at(b + 64).row : -1;  // first row of the next step
    v = scan_sum_by_key(v, row);
    int next = __shfl_down(row, 1, 64);
    if (lane == 63) next = after;
    const float total = v + (row == carry_row ? carry : 0.f);
    if (ok && next != row) finish(row, total);
    const int row63 = __builtin_amdgcn_readlane(row, 63);
    const float tot63 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(total), 63));
    const bool runs_on = row63 >= 0 && after == row63;
    carry_row = runs_on ? row63 : -1;
    carry = runs_on ? tot63 : 0.f;
  }
}

// The thread's number.  HIDE: unknown to the compiler at the places where it is asked for, so that
// addresses made from it are worked out again in every phase of an epoch.  Known, they are all made
// ahead of the loop over the epochs, and held in registers across it they and others spill (three
// layers of width 32: 75 registers, 33 with this), each reload waiting for every load in flight:
// 256 subgraphs of 200 rows of width 32, three layers, 47.6 -> 43.9 us per epoch, of 128 rows of width
// 64 65.2 -> 60.9.  Two layers of width 8 or 16 spill twelve at most, and working the addresses out costs
// more (200 rows: 14.3 us against 15.0).
template <bool HIDE>
__device__ __forceinline__ int thread_number() {
  int tid = threadIdx.x;
  if (HIDE) asm volatile("" : "+v"(tid));
  return tid;
}

// Backward of hidden layer l (see BwdArgs), then Adam on W_l (and on w_out by the last layer).
template <typename T, int D, int L, bool GRADS, bool LAST, bool TO_EMBED>
__device__ __forceinline__ void backward_layer(const SmallTrain& a, const StreamInLds& st, const GraphView& g, float* smem,
                               const Carve<D>& cv, const int k, const int R, const size_t first, const AdamStep& adE,
                               const AdamStep& adW) {
  using K = SK<D>;
  constexpr int NQ = K::NQ, DP = K::DP, PT = K::PT, NW = K::NW, WP = K::WP;
  constexpr int l = LAST ? L - 1 : 1;
  static_assert(TO_EMBED == (l == 1), "the layer's number");
  using Rows = std::conditional_t<LAST, LastRows<D, T>, PlainRows<D, T>>;
  const int tid = thread_number<(L == 3 || D >= 32)>(), lane = tid % 64, n = lane % 16, h = lane / 16;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  float* gt = smem + cv.sums + wave * K::kWaveLds;
  float* wl = smem + cv.w[l - 1];
  const T* Hprev = static_cast<const T*>(a.H[l - 1]) + first * D;
  Rows rows;
  if constexpr (LAST) {
    rows.H = static_cast<const T*>(a.H[l]) + first * D;
    rows.g_t = smem + cv.p;  // g_t has taken the place of p
#pragma unroll
    for (int q = 0; q < NQ; ++q) rows.w[q] = *reinterpret_cast<const f32x4*>(smem + cv.wo + 16 * q + 4 * (lane % 4));
  } else {
    rows.X = static_cast<const T*>(a.GZ) + first * D;
  }
  f32x4 gw[NQ][NQ], gwo[LAST ? NQ : 1];
#pragma unroll
  for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
    for (int tb = 0; tb < NQ; ++tb) gw[ta][tb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int q = 0; q < (LAST ? NQ : 1); ++q) gwo[q] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int r0 = wave * kTile; r0 < R; r0 += NW * kTile) {
    const int row = r0 + n, safe = min(row, R - 1);
    // rows of Hprev as the A operand of the weight gradient
    float av[4][NQ];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int ta = 0; ta < NQ; ++ta) {
        const int hr = r0 + 4 * s + h;
        av[s][ta] = hr < R && (D >= 16 || n < D) ? Store<T>::get(Hprev + static_cast<size_t>(hr) * D + 16 * ta + n) : 0.f;
      }
    TileFacts<D> f;
    f.request(st, r0, R);
    f.request_entries(st);
    f32x4 acc[NQ];
    aggregate<D>(g, st, rows, f, r0, R, nullptr, gt, acc, [&](const typename Rows::Row& own) {
      if constexpr (LAST) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int y = 0; y < 4; ++y) gwo[q][y] = fmaf(own.x[q][y], own.gt, gwo[q][y]);
      }
    });
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
#pragma unroll
      for (int y = 0; y < 4; ++y) acc[q][y] = Store<T>::as_stored(acc[q][y]);
      *reinterpret_cast<f32x4*>(gt + n * PT + 16 * q + 4 * h) = acc[q];
    }
    wave_lds_handoff();
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float bv[NQ];
#pragma unroll
      for (int tb = 0; tb < NQ; ++tb) bv[tb] = gt[(4 * s + h) * PT + 16 * tb + n];
#pragma unroll
      for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
        for (int tb = 0; tb < NQ; ++tb) gw[ta][tb] = mfma(av[s][ta], bv[tb], gw[ta][tb]);
    }
    wave_lds_handoff();
    if (TO_EMBED && (GRADS ? a.gE == nullptr : !a.train_embed)) continue;
    const int on = operand_lane<D>(n);
#pragma unroll
    for (int ta = 0; ta < NQ; ++ta) {
      f32x4 e, m, v;
      if (TO_EMBED) {
        e = load4<D>(a.E + first * D, safe, ta, h);
        m = load4<D>(a.mE + first * D, safe, ta, h);
        v = load4<D>(a.vE + first * D, safe, ta, h);
      } else {
        e = load4<D>(Hprev, safe, ta, h);
      }
      f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        const f32x4 w = *reinterpret_cast<const f32x4*>(wl + (16 * ta + on) * WP + 16 * q + 4 * h);
#pragma unroll
        for (int j = 0; j < 4; ++j) z = mfma(w[j], acc[q][j], z);
      }
      if (row < R) {
        if constexpr (TO_EMBED && GRADS) {
          store4<D>(a.gE + first * D, row, ta, h, z);
        } else if constexpr (TO_EMBED) {
          adam_rows(adE, z, e, m, v);
          store4<D>(a.mE + first * D, row, ta, h, m);
          store4<D>(a.vE + first * D, row, ta, h, v);
          store4<D>(a.E + first * D, row, ta, h, e);
          if constexpr (sizeof(T) == 2) store4<D>(static_cast<T*>(a.Eb) + first * D, row, ta, h, e);
        } else {
#pragma unroll
          for (int x = 0; x < 4; ++x) z[x] = e[x] > 0.f ? z[x] : 0.f;
          store4<D>(static_cast<T*>(a.GZ) + first * D, row, ta, h, z);
        }
      }
    }
  }

  // the wavefronts' sums of the weight gradient, in order, and Adam on W_l
  if constexpr (LAST) {
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int y = 0; y < 4; ++y) {
        const float s = groups_sum(gwo[q][y]);
        if (lane < 4) smem[cv.gwo + wave * DP + 16 * q + 4 * lane + y] = s;
      }
  }
  __syncthreads();  // the row sums have served
  constexpr bool kHalves = DP * DP > K::kWaveLds;  // the place holds half the wavefronts' sums
  constexpr int kSlots = kHalves ? NW / 2 : NW;
  static_assert(kSlots * DP * DP <= NW * K::kWaveLds, "room for the sums");
  float* slots = smem + cv.sums;
  auto each = [&](auto&& fn) {
    float* mine = slots + (wave % kSlots) * DP * DP;
#pragma unroll
    for (int ta = 0; ta < NQ; ++ta)
#pragma unroll
      for (int tb = 0; tb < NQ; ++tb)
#pragma unroll
        for (int r = 0; r < 4; ++r) fn(mine[(16 * ta + 4 * h + r) * DP + 16 * tb + n], gw[ta][tb][r]);
  };
  if (wave >= NW - kSlots) each([](float& place, float x) { place = x; });
  __syncthreads();
  if (kHalves) {
    if (wave < kSlots) each([](float& place, float x) { place = x + place; });
    __syncthreads();
  }
  if constexpr (GRADS) {
    for (int idx = tid; idx < D * D; idx += K::NT) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < kSlots; ++q) s += slots[q * DP * DP + idx / D * DP + idx % D];
      a.gW[l - 1][static_cast<size_t>(k) * D * D + idx] = s;
    }
    if (LAST && tid < D) {
      float s = 0.f;
#pragma unroll
      for (int q = 0; q < NW; ++q) s += smem[cv.gwo + q * DP + tid];
      a.gW[L - 1][static_cast<size_t>(k) * D + tid] = s;
    }
    __syncthreads();
    return;
  }
  float* W = a.W[l - 1] + static_cast<size_t>(k) * D * D;
  float* mW = a.mW[l - 1] + static_cast<size_t>(k) * D * D;
  float* vW = a.vW[l - 1] + static_cast<size_t>(k) * D * D;
  for (int idx = tid; idx < D * D; idx += K::NT) {
    const int r = idx / D, c = idx % D;
    float w = W[idx], m = mW[idx], v = vW[idx], s = 0.f;
#pragma unroll
    for (int q = 0; q < kSlots; ++q) s += slots[q * DP * DP + r * DP + c];
    adam_value(adW, s, w, m, v);
    W[idx] = w;
    mW[idx] = m;
    vW[idx] = v;
    wl[r * WP + c] = Store<T>::as_stored(w);
  }
  if (LAST && tid < D) {
    const size_t idx = static_cast<size_t>(k) * D + tid;
    float w = a.W[L - 1][idx], m = a.mW[L - 1][idx], v = a.vW[L - 1][idx], s = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) s += smem[cv.gwo + q * DP + tid];
    adam_value(adW, s, w, m, v);
    a.W[L - 1][idx] = w;
    a.mW[L - 1][idx] = m;
    a.vW[L - 1][idx] = v;
    smem[cv.wo + tid] = w;
  }
  __syncthreads();
}

// Copies the weight sets of subgraph k to the snapshot.
template <int D, int L>
__device__ __forceinline__ void keep_weights(const SmallTrain& a, int k) {
#pragma unroll
  for (int l = 0; l < L; ++l) {
    const int elems = l < L - 1 ? D * D : D;
    for (int i = threadIdx.x; i < elems; i += SK<D>::NT)
      a.W_best[l][static_cast<size_t>(k) * elems + i] = a.W[l][static_cast<size_t>(k) * elems + i];
  }
}

// What a launch is for; each is compiled by itself.  Training does not carry the gradients' stores, and
// forward and loss not the registers of the backward pass (which spill, so that a launch of its own started
// later: 512 subgraphs of 60 rows of width 16, forward 17.6 -> 11.2 us).
enum class Purpose { kForward, kTrain, kGradients };  // passes 1 and 2; 3; 4

template <typename T, int D, int L, Purpose FOR>
__global__ __launch_bounds__(SK<D>::NT) void small_train_kernel(GraphView g, SmallTrain a) {
  using K = SK<D>;
  constexpr int NQ = K::NQ, DP = K::DP, NW = K::NW, NT = K::NT, WP = K::WP;
  extern __shared__ __align__(16) float smem[];
  const int k = blockIdx.x;
  if (g.loss_ptr[k + 1] == g.loss_ptr[k]) return;  // the subgraph sits out
  const int rbeg = g.part_rows[k], R = g.part_rows[k + 1] - rbeg;
  if (R == 0) {  // no rows: a loss of nothing
    if (a.passes == 1) return;
    if constexpr (FOR == Purpose::kGradients) {
#pragma unroll
      for (int l = 0; l < L; ++l) {
        const int elems = l < L - 1 ? D * D : D;
        for (int i = threadIdx.x; i < elems; i += NT) a.gW[l][static_cast<size_t>(k) * elems + i] = 0.f;
      }
      return;
    }
    for (int ep = threadIdx.x; ep < a.epochs; ep += NT) a.loss_partial[static_cast<size_t>(ep) * g.num_loss_slots + k] = 0.0;
    if (a.best_loss != nullptr && a.best_loss[k] > 0.0) {  // its one model, whose loss is 0 from the first epoch on
      __syncthreads();
      keep_weights<D, L>(a, k);
      if (threadIdx.x == 0) {
        a.best_loss[k] = 0.0;
        a.has_best[k] = 1;
      }
    }
    return;
  }
  const size_t first = rbeg;
  const bool mean = g.wval != g.wval_t;
  const int es = g.wrowptr[rbeg], En = g.wrowptr[rbeg + R] - es;
  const Carve<D> cv(L, R, En, mean);
  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
  int* rp = reinterpret_cast<int*>(smem + cv.rp);
  uint2* ent = reinterpret_cast<uint2*>(smem + cv.ent);
  double* dred = reinterpret_cast<double*>(smem + cv.red);
  double* lowest = dred + NW;
  int* lower = reinterpret_cast<int*>(lowest + 1);

  for (int i = tid; i <= R; i += NT) rp[i] = g.wrowptr[rbeg + i] - es;
  for (int i = tid; i < R; i += NT) smem[cv.c + i] = a.c[rbeg + i];
  for (int e = tid; e < En + kSmallPad; e += NT) {
    uint2 x = make_uint2(0u, 0u);
    if (e < En) {
      x.x = static_cast<uint32_t>(g.went[es + e].x - rbeg) | static_cast<uint32_t>(g.wrowid[es + e] - rbeg) << 16;
      x.y = __float_as_uint(g.wval[es + e]);
    }
    ent[e] = x;
    if (mean) smem[cv.valt + e] = e < En ? g.wval_t[es + e] : 0.f;
  }
#pragma unroll
  for (int l = 1; l < L; ++l)
    for (int idx = tid; idx < DP * DP; idx += NT) {
      const int r = idx / DP, c = idx % DP;
      smem[cv.w[l - 1] + r * WP + c] =
          r < D && c < D ? Store<T>::as_stored(a.W[l - 1][static_cast<size_t>(k) * D * D + r * D + c]) : 0.f;
    }
  if (tid < DP) smem[cv.wo + tid] = tid < D ? a.W[L - 1][static_cast<size_t>(k) * D + tid] : 0.f;
  if (tid == 0) *lowest = a.best_loss != nullptr ? a.best_loss[k] : 0.0;
  __syncthreads();
  const StreamInLds fwd{ent, nullptr, rp};
  const StreamInLds bwd{ent, mean ? smem + cv.valt : nullptr, rp};

  // width-1 phases: whole rows of this wavefront, cut at equal shares of the entries
  auto first_row_from = [&](int e) {
    int lo = 0, hi = R;  // the first row whose entries begin at e or later
    while (lo < hi) {
      const int mid = (lo + hi) / 2;
      if (rp[mid] >= e) hi = mid; else lo = mid + 1;
    }
    return lo;
  };
  const int e0 = rp[first_row_from(static_cast<int>(static_cast<int64_t>(En) * wave / NW))];
  const int e1 = rp[first_row_from(static_cast<int>(static_cast<int64_t>(En) * (wave + 1) / NW))];
  float *tv = smem + cv.t, *pv = smem + cv.p;

  for (int ep = 0; ep < a.epochs; ++ep) {
    const int tid = thread_number<(L == 3 || D == 64)>(), lane = tid % 64, n = lane % 16, h = lane / 16;
    AdamStep adE = a.adam, adW = a.adam;
    if (a.adam.per_part != nullptr) {
      const float2* bc = a.adam.per_part + static_cast<size_t>(ep) * (2 * g.P);  // [P] embeddings, [P] weights
      adE.inv_bc1 = bc[k].x;
      adE.inv_sqrt_bc2 = bc[k].y;
      adW.inv_bc1 = bc[g.P + k].x;
      adW.inv_sqrt_bc2 = bc[g.P + k].y;
    } else {
      adE.inv_bc1 = adW.inv_bc1 = a.bc[ep].x;
      adE.inv_sqrt_bc2 = adW.inv_sqrt_bc2 = a.bc[ep].y;
    }
    // hidden layers of Eq. 3; the last one also leaves t = H w_out
#pragma unroll
    for (int l = 1; l < L; ++l) {
      const PlainRows<D, T> rows{static_cast<const T*>(a.H[l - 1]) + first * D};
      T* Y = static_cast<T*>(a.H[l]) + first * D;
      const float* wl = smem + cv.w[l - 1];
      float* sums = smem + cv.sums + wave * K::kWaveLds;
      for (int r0 = wave * kTile; r0 < R; r0 += NW * kTile) {
        const int row = r0 + n;
        TileFacts<D> f;
        f.request(fwd, r0, R);
        f.request_entries(fwd);
        f32x4 acc[NQ];
        aggregate<D>(g, fwd, rows, f, r0, R, nullptr, sums, acc, [](const typename PlainRows<D, T>::Row&) {});
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int y = 0; y < 4; ++y) acc[q][y] = Store<T>::as_stored(acc[q][y]);
        float part = 0.f;
        const int on = operand_lane<D>(n);
#pragma unroll
        for (int ta = 0; ta < NQ; ++ta) {
          f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) z = mfma(wl[(16 * q + 4 * h + j) * WP + 16 * ta + on], acc[q][j], z);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            z[j] = Store<T>::as_stored(fmaxf(z[j], 0.f));
            if (l == L - 1) part = fmaf(z[j], smem[cv.wo + 16 * ta + 4 * h + j], part);
          }
          if (row < R) store4<D>(Y, row, ta, h, z);
        }
        if (l == L - 1) {
          part += __shfl_xor(part, 16, 64);
          part += __shfl_xor(part, 32, 64);
          if (h == 0 && row < R) tv[row] = part;
        }
      }
      __syncthreads();
    }
    // Eq. 4, the loss of Eq. 5 with its derivative, and the first backward aggregation
    const bool keep_p = ep == a.epochs - 1;
    scan_rows(fwd, e0, e1, [&](const Entry& en) { return en.val * tv[en.col]; },
              [&](int row, float s) {
                const float p = 1.f / (1.f + expf(-s));
                pv[row] = p;
                if (keep_p) a.p[rbeg + row] = p;
              });
    if (FOR == Purpose::kForward && a.passes == 1) return;
    __syncthreads();
    double lsum = 0.0;
    scan_rows(fwd, e0, e1, [&](const Entry& en) { return en.col == en.row ? 0.f : pv[en.col]; },
              [&](int row, float s) {
                const float p = pv[row], c = smem[cv.c + row];
                tv[row] = (c + a.q * s) * p * (1.f - p);
                lsum += static_cast<double>(p) *
                        (static_cast<double>(c) + 0.5 * static_cast<double>(a.q) * static_cast<double>(s));
              });
    lsum = wave_sum(lsum);
    if (lane == 0) dred[wave] = lsum;
    __syncthreads();
    if (tid == 0) {
      double total = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) total += dred[w];
      a.loss_partial[static_cast<size_t>(ep) * g.num_loss_slots + k] = total;
      *lower = a.best_loss != nullptr && total < *lowest;
      if (*lower) {
        *lowest = total;
        a.best_loss[k] = total;
        a.has_best[k] = 1;
      }
    }
    if constexpr (FOR == Purpose::kForward) {
      return;
    } else {
    scan_rows(bwd, e0, e1, [&](const Entry& en) { return en.val * tv[en.col]; },
              [&](int row, float s) { pv[row] = s; });
    __syncthreads();
    if (*lower) {  // the parameters this loss belongs to, before they change
      const float4* from = reinterpret_cast<const float4*>(a.E + first * D);
      float4* to = reinterpret_cast<float4*>(a.E_best + first * D);
      for (int i = tid; i < R * (D / 4); i += NT) to[i] = from[i];
      keep_weights<D, L>(a, k);
      __syncthreads();
    }
    constexpr bool kGrads = FOR == Purpose::kGradients;
    if constexpr (L == 2) {
      backward_layer<T, D, L, kGrads, true, true>(a, bwd, g, smem, cv, k, R, first, adE, adW);
    } else {
      backward_layer<T, D, L, kGrads, true, false>(a, bwd, g, smem, cv, k, R, first, adE, adW);
      backward_layer<T, D, L, kGrads, false, true>(a, bwd, g, smem, cv, k, R, first, adE, adW);
    }
    }
  }
}

template <typename T, int D, int L>
void launch_t(const Launch& ln, const GraphView& g, const SmallTrain& a, size_t lds) {
  auto run = [&](auto kernel) {
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              static_cast<int>(lds));
    kernel<<<g.P, SK<D>::NT, lds, ln.st>>>(g, a);
  };
  if (a.passes <= 2) run(small_train_kernel<T, D, L, Purpose::kForward>);
  else if (a.passes == 3) run(small_train_kernel<T, D, L, Purpose::kTrain>);
  else run(small_train_kernel<T, D, L, Purpose::kGradients>);
}

template <typename T, int D>
void launch_l(const Launch& ln, int L, const GraphView& g, const SmallTrain& a, size_t lds) {
  if (L == 2) launch_t<T, D, 2>(ln, g, a, lds);
  else if (L == 3) launch_t<T, D, 3>(ln, g, a, lds);
}

}  // namespace

size_t small_train_lds_bytes(int D, int L, int rows, int entries, bool mean) {
  size_t floats = 0;
  switch (D) {
    case 8: floats = Carve<8>(L, rows, entries, mean).end; break;
    case 16: floats = Carve<16>(L, rows, entries, mean).end; break;
    case 32: floats = Carve<32>(L, rows, entries, mean).end; break;
    case 64: floats = Carve<64>(L, rows, entries, mean).end; break;
    default: return static_cast<size_t>(-1);
  }
  return floats * sizeof(float);
}

void launch_small_train(const Launch& ln, int storage, int D, int L, const GraphView& g, const SmallTrain& a,
                        size_t lds) {
  ln.begin(KK_SMALL_TRAIN);
  if (storage == GCO_STORAGE_BF16) {
    if (D == 64) launch_l<bf16_t, 64>(ln, L, g, a, lds);
  } else if (D == 8) {
    launch_l<float, 8>(ln, L, g, a, lds);
  } else if (D == 16) {
    launch_l<float, 16>(ln, L, g, a, lds);
  } else if (D == 32) {
    launch_l<float, 32>(ln, L, g, a, lds);
  } else if (D == 64) {
    launch_l<float, 64>(ln, L, g, a, lds);
  }
  ln.end(KK_SMALL_TRAIN);
}

}  // namespace gco
