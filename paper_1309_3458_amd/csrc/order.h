// The order that updates are matched in (d > 1): what a sample of them decides
// about the whole set (probe dimensions, cells, whether the set is dense), and the
// cell of every update.  Shared by the single-instance and the batched matcher.
#pragma once

#include "traverse.h"

namespace ddm {

// updates per tile: 64, or fewer (down to one) while that leaves at most
// kFewTiles tiles, so that the chip has wavefronts to run and few updates in a
// large set do not share boxes wider than their own (17,389 updates of 21 hits
// each, count: 73 us with 16 to a tile, 21 with 4; 1100 updates against 490,000
// subscriptions: d = 4 563 us with 4, 22 with one, d = 3 165 and 10, d = 1 51
// and 9)
constexpr uint32_t kFewTiles = 8192;
__host__ __device__ inline uint32_t tile_updates(uint32_t m) {
  uint32_t q = 1;
  while (q < 64u && m > q * kFewTiles) q *= 2;
  return q;
}

// Quantiles held in LDS are padded by one word after every 64: the lanes of
// a binary search read indices a power of two apart, which without padding
// fall into one LDS bank at the middle levels of the search.
constexpr uint32_t kQuantPad = kQuant + kQuant / 64;
__device__ __forceinline__ uint32_t qslot(uint32_t i) { return i + (i >> 6); }

// the probe estimate of an update: the probe dimension bk, #quantiles <=
// q.hi and < q.lo - maxlen there (bqa, bqb), #quantiles <= the box centre in
// every dimension, and whether the extent is invalid
template <int D>
struct ProbeEst {
  uint32_t bk, bqa, bqb;
  uint32_t mid[D];
  uint32_t est[D];  // quantiles of the candidate positions in every dimension
  float hits;  // subscriptions met, were the dimensions independent
  bool bad;
};

// the update's extents (ua, ub: dimension k of update j), loaded before the
// quantiles are (their loads overlap)
template <int D>
struct UpdExt {
  float a[D], b[D];
};
template <int D>
__device__ __forceinline__ UpdExt<D> load_ext(const float* __restrict__ ulo,
                                              const float* __restrict__ uhi, uint32_t m,
                                              uint32_t j) {
  UpdExt<D> e;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    e.a[k] = ulo[(size_t)k * m + j];
    e.b[k] = uhi[(size_t)k * m + j];
  }
  return e;
}

// the kQuant quantiles of every dimension into LDS (sq[k][qslot(i)]), by
// THREADS threads: every load is issued before the first LDS store, so that
// they are in flight together
template <int D, uint32_t THREADS>
__device__ __forceinline__ void load_quant_lds(const TreeDev& T, uint32_t (*sq)[kQuantPad]) {
  static_assert(kQuant % THREADS == 0, "whole rounds");
  constexpr uint32_t Q = kQuant / THREADS;
  uint32_t v[D][Q];
#pragma unroll
  for (int k = 0; k < D; ++k)
#pragma unroll
    for (uint32_t r = 0; r < Q; ++r) v[k][r] = T.quant[k][r * THREADS + threadIdx.x];
#pragma unroll
  for (int k = 0; k < D; ++k)
#pragma unroll
    for (uint32_t r = 0; r < Q; ++r) sq[k][qslot(r * THREADS + threadIdx.x)] = v[k][r];
}

// The class of an update is its probe dimension: one for the whole set (the
// dimension whose ranges are the shortest on average), or every update's own
// (kOwnClass), for small sets, the lane form, and where a second dimension holds a
// real share.  With own classes the few updates of a set that leave the common
// one make up tiles that span the space: the 16-hotspot workload, ten seeds, 6.5 ..
// 9.4 ms, mean 7.5, against 6.5 .. 7.3, mean 6.8; d = 4, 62,266 updates, a count of
// 284 us against 84.  With one class where half of the updates are long in the one
// dimension and half in the other, every tile is long in both (100,000 updates, 0.2
// of the space by 20 units, against 250,000 squares: match 694 us, own classes 126).
// So the set has one class unless that makes its ranges kClassCost times as long as
// the updates' own would be (hotspots: up to 1.15, equal boxes 1, that set 2 to 400).
constexpr uint32_t kOwnClass = ~0u;
constexpr float kClassCost = 1.5f;

// len (may be null): the lengths of a subscription, which the hits are then for, as
// the ranges are for the longest ones
template <int D>
__device__ __forceinline__ ProbeEst<D> probe_estimate(const TreeDev& T,
                                                      const uint32_t (*sq)[kQuantPad],
                                                      const UpdExt<D>& e, uint32_t cls,
                                                      const float* len = nullptr) {
  ProbeEst<D> P;
  P.bad = false;
  uint32_t xh[D], xl[D], xm[D], xs[D], qa[D], qb[D], qm[D], qs[D];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const float a = e.a[k], b = e.b[k];
    P.bad = P.bad || !valid_extent(a, b);
    xh[k] = f2key(b);
    xl[k] = f2key(nextafterf(a - T.maxlen[k], -INFINITY));
    xm[k] = f2key(0.5f * a + 0.5f * b);
    xs[k] = len ? f2key(nextafterf(a - len[k], -INFINITY)) : 0u;
    qa[k] = qb[k] = qm[k] = qs[k] = 0;
  }
  // the 3D quantile searches (#quantiles <= xh, < xl, <= xm per dimension; 4D with
  // len) advance in lockstep, so their LDS reads overlap
#pragma unroll
  for (uint32_t step = kQuant; step > 0; step >>= 1) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const uint32_t ca = qa[k] + step, cb = qb[k] + step, cm = qm[k] + step;
      const uint32_t va = ca <= kQuant ? sq[k][qslot(ca - 1)] : 0xffffffffu;
      const uint32_t vb = cb <= kQuant ? sq[k][qslot(cb - 1)] : 0xffffffffu;
      const uint32_t vm = cm <= kQuant ? sq[k][qslot(cm - 1)] : 0xffffffffu;
      if (ca <= kQuant && va <= xh[k]) qa[k] = ca;
      if (cb <= kQuant && vb < xl[k]) qb[k] = cb;
      if (cm <= kQuant && vm <= xm[k]) qm[k] = cm;
      if (len) {
        const uint32_t cs = qs[k] + step;
        const uint32_t vs = cs <= kQuant ? sq[k][qslot(cs - 1)] : 0xffffffffu;
        if (cs <= kQuant && vs < xs[k]) qs[k] = cs;
      }
    }
  }
  // an update's own class: dimension 0, unless another one's range is less than
  // a third as long (at the edge of the space a range is half as long)
  uint32_t best = 0;
  P.hits = (float)T.n;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const uint32_t est = qa[k] - min(qa[k], qb[k]);
    const uint32_t meets = len ? qa[k] - min(qa[k], qs[k]) : est;
    P.hits *= fmaxf((float)meets, 0.5f) * (1.f / (float)kQuant);
    P.mid[k] = qm[k];
    P.est[k] = est;
    if (cls == kOwnClass ? k == 0 || 3u * est + 16u < best : (uint32_t)k == cls) {
      best = est;
      P.bk = (uint32_t)k;
      P.bqa = qa[k];
      P.bqb = qb[k];
    }
  }
  return P;
}

// What the sample decides.  The rows of b are the classes; one class for the set
// has the cells of all.
struct OrderPlan {
  uint32_t cls;                     // the set's class, or kOwnClass
  uint32_t b[DDM_MAX_D][DDM_MAX_D]; // cells along the class's own dimension, then the others
};

constexpr uint32_t kPlanThreads = 1024, kPlanSamples = 256;
constexpr uint32_t kQuantLog = 12;
static_assert(1u << kQuantLog == kQuant, "quantiles are counted in so many bits");

// Sets whose dimensions depend on each other (extents along a line or a plane, or in
// clusters) fill few cells of a grid, and the updates of a cell come in no order, so
// that every tile is as wide as its cell.  How crowded the cells are shows in the
// pairs of samples that share one: their share of all pairs is that of a cell's
// candidates among the subscriptions.  Where it is more than twice a tile's and
// not by chance (kCrowdedPairs), grids that are finer in the class's own dimension
// are tried, and the finest taken that reads as little as any (within kFinerSlack:
// the largest tile is the smaller, the finer it is).  Candidates of a tile on
// average, 500,000 + 500,000 boxes, first grid / own dimension 4, 16 and 64 times
// finer / every quantile:
//   along a line, d = 3         12,234 / 5749 / 1562 / 443 / 189
//   16 clusters,  d = 2            199 /  217 /  291 /   - / 511
//                 d = 3           1310 / 1176 /  767 / 760 / 1043
//                 d = 4           2995 / 2772 / 1355 / 675 / 1130
//   uniform,      d = 4 (200,000)   71 /   92 /  194 / 554 / 4496
// Match, us, before there were such grids / first grid / now: a line of 500,000,
// d = 2 303/886/298, d = 3 236/4507/226, d = 4 260/8845/245; a plane, d = 4, 200,000
// 205/3120/210; 100 clusters, d = 3 269/530/228.
constexpr uint32_t kCrowdedPairs = 20, kFinest = 4;
constexpr float kFinerSlack = 1.3f;
constexpr uint32_t kSeen = 16384;  // counters of samples in a cell (16 bits each)

// Cells of a class of m updates whose ranges are r quantile steps long on average:
// along each dimension, the class's own first and the others ascending.  A tile of
// width w reads what meets w + r, and its widths multiply to the same volume
// whatever the shape, so that the sum is least where widths go with ranges: all
// dimensions but the last are cut into as many ranges as there are tiles of 64
// along one, more where ranges are shorter than their mean, the last into as many
// as the rest of the `cells` allow, so that a tile takes a few cells of one line.
// (250,000 + 250,000 boxes, half 60,000 long in the one and half in the other of
// two dimensions, 3000 in the third: match 383 us with the same cut in all, 315 now.)
// finer > 0: 4^finer as many ranges along the class's own dimension (the last
// step: every quantile), and what is left over the others.
// Returns the share of the space that a tile reads, in volumes of a cell.
template <int D>
__device__ __forceinline__ float cell_shape(float m, uint32_t cls, uint32_t cells,
                                            const float (&r)[D], uint32_t finer,
                                            uint32_t (&b)[DDM_MAX_D]) {
  float lg[D], mean = 0.f, own = 0.f;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    lg[k] = log2f(fmaxf(r[k], 1.f));
    mean += lg[k] / (float)D;
    if ((uint32_t)k == cls) own = lg[k];
  }
  const float along = log2f(m / 64.f) / (float)D;
  const float others = (mean * (float)D - own) / (float)(D - 1);  // their mean
  uint32_t rest = cells;
  float reads = 1.f, left = 0.f;
#pragma unroll
  for (int s = 0; s < DDM_MAX_D; ++s) {
    if (s >= D) {
      b[s] = 1;
      continue;
    }
    const uint32_t kk = s == 0 ? cls : (uint32_t)(s - 1) + (((uint32_t)(s - 1) >= cls) ? 1u : 0u);
    float l = 0.f;
#pragma unroll
    for (int k = 0; k < D; ++k)
      if ((uint32_t)k == kk) l = lg[k];
    float want = along + mean - l;
    if (finer) {
      if (s == 0) want = finer < kFinest ? want + 2.f * (float)finer : (float)kQuantLog;
      else want = left + others - l;
    }
    const uint32_t most = s == 0 ? min(rest, kQuant) : max(rest / 2u, 1u);
    b[s] = max(1u, s + 1 < D ? min((uint32_t)(exp2f(want) + 0.5f), finer ? most : rest / 2u)
                             : rest);
    rest /= b[s];
    if (s == 0) left = log2f((float)rest) / (float)(D - 1);
    reads *= 1.f + exp2f(l - (float)kQuantLog) * (float)min(b[s], kQuant);
  }
  return reads;
}

// the cell of an update of class c on the grid b (its row), from the quantiles
// below its centre; the numbering is a serpentine (each line runs back where the
// last one ended)
template <int D>
__device__ __forceinline__ uint32_t grid_cell(const uint32_t* __restrict__ b, uint32_t c,
                                              const uint32_t (&mid)[D]) {
  uint32_t sub = 0;
#pragma unroll
  for (int s = 0; s < D; ++s) {
    const uint32_t kk = s == 0 ? c : (uint32_t)(s - 1) + (((uint32_t)(s - 1) >= c) ? 1u : 0u);
    uint32_t qp = 0;
#pragma unroll
    for (int k = 0; k < D; ++k)
      if ((uint32_t)k == kk) qp = mid[k];
    const uint32_t n = b[s];
    uint32_t i = min(qp * n / (kQuant + 1u), n - 1u);
    if (sub & 1u) i = n - 1u - i;  // the serpentine's way back
    sub = sub * n + i;
  }
  return sub;
}

// Up to kPlanSamples updates spread evenly over the set decide whether the
// count traversal keeps its hits: the stash is marked full before it is used,
// and the set matched as a dense one, when the estimated hits (the candidate
// fractions of the dimensions multiplied, as if they were independent, with the
// lengths of a sample of subscriptions) exceed four fifths of the stash's counted chunks (tiles leave some of theirs), or per
// update the larger of kDenseHits and
// kDenseScale * d / sqrt(m).  The dense form takes two more synchronizations and
// nine more launches, a fixed 70 us, and saves on every pair, the more the more
// updates lie near each other.  Match of m updates against m subscriptions, us,
// keeping hits / dense form (10, 20, 40, 80 hits each):
//   d = 2  m =  20,000   86/157   91/158  138/157  232/152
//          m =  80,000  128/164  164/159  306/164  345/173
//          m = 250,000  240/229  388/236  530/245  603/273
//   d = 3  m =  20,000   92/160  101/169  146/170  184/178
//          m =  80,000  145/189  181/199  370/211  492/251
//   d = 4  m =  80,000  208/283  211/305  505/369  731/424
// A set whose dimensions are correlated may still overflow the stash.
constexpr float kDenseHits = 10.f, kDenseScale = 3000.f;

// LDS of the sample, beside the quantiles
template <int D>
struct SampleLds {
  static constexpr int kWaves = kPlanSamples / kWave;
  uint32_t part[D * (D + 1)][kWaves];  // sums of the wavefronts
  float hits[kWaves];
  uint32_t sum[D * (D + 1)];
  float total;
  uint32_t b[D][DDM_MAX_D];
  float reads[D];
  uint32_t pairs;
};

// adds up `count` values of part and the hits
template <int D>
__device__ __forceinline__ void sample_sums(SampleLds<D>& L, uint32_t count) {
  constexpr uint32_t W = SampleLds<D>::kWaves;
  __syncthreads();
  if (threadIdx.x < count) {
    uint32_t s = 0;
    for (uint32_t w = 0; w < W; ++w) s += L.part[threadIdx.x][w];
    L.sum[threadIdx.x] = s;
  }
  if (threadIdx.x == kWave) {
    float t = 0.f;
    for (uint32_t w = 0; w < W; ++w) t += L.hits[w];
    L.total = t;
  }
  __syncthreads();
}

// Run by one workgroup of kPlanThreads; the first kPlanSamples of them take a
// sample each (1024 samples took 5 us longer at d = 2, 10 at d = 4: one compute
// unit does the searches).  full (may be null):
// where the stash is marked, with mark (kStashDense where the dense form may
// follow, else 1, a stash that is full, so that the count traversal counts at
// once).  plan (may be null): cells to a class, q updates to a tile; lanes: for the
// lane form, classes of their own whatever the ranges, and the finest cells along the
// own dimension, the only one that a lane's walk depends on (100,000 updates, count
// and fill by lanes, d = 2 2304 us with the cells of the tiles, 1764 with these,
// d = 3 17,010 and 12,210).  (sq is overwritten.)
template <int D>
__device__ __forceinline__ void sample_set(const TreeDev& T, const float* __restrict__ ulo,
                                           const float* __restrict__ uhi, uint32_t m,
                                           uint32_t (*sq)[kQuantPad], SampleLds<D>& L,
                                           uint32_t* __restrict__ full, uint32_t mark,
                                           uint32_t room, OrderPlan* __restrict__ plan,
                                           uint32_t cells, uint32_t q, bool lanes) {
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const uint32_t S = min(m, kPlanSamples);
  UpdExt<D> e{};
  if (tid < S) e = load_ext<D>(ulo, uhi, m, (uint32_t)(((uint64_t)tid * m) / S));
  // a subscription for each sample, at even positions of a tree: were all as long as
  // the longest, 250,000 + 250,000 boxes, half 60,000 long in the one and half in the
  // other of two dimensions, 3.3 hits each, would count as dense (match 318 us, 178 now)
  float rec[2 * D] = {};
  if (tid < S)
    load_rec<D>(T.rec[0] + (size_t)(1u + (uint32_t)(((uint64_t)tid * T.n) / S)) * 2 * D, rec);
  load_quant_lds<D, kPlanThreads>(T, sq);
  __syncthreads();
  ProbeEst<D> P{};
  bool in = tid < S;
  if (tid < kPlanSamples) {
    if (in) {
      float len[D];
#pragma unroll
      for (int k = 0; k < D; ++k) len[k] = nextafterf(rec[2 * k + 1] - rec[2 * k], INFINITY);
      P = probe_estimate<D>(T, sq, e, kOwnClass, len);
      in = !P.bad;
    }
    float hits = in ? P.hits : 0.f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) hits += __shfl_xor(hits, o, kWave);
    uint32_t mine = 0;  // the range in the sample's own class
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const uint32_t v = wave_scan_dpp(in ? P.est[k] : 0u);
      if (lane == kWave - 1) L.part[k][wave] = v;
      if ((uint32_t)k == P.bk) mine = P.est[k];
    }
    const uint32_t v = wave_scan_dpp(in ? mine : 0u);
    if (lane == kWave - 1) L.part[D][wave] = v;
    if (lane == 0) L.hits[wave] = hits;
  }
  sample_sums(L, D + 1);
  if (tid == 0 && full) {
    const float t = L.total / (float)S;
    const float dense = fmaxf(kDenseHits, kDenseScale * (float)D * rsqrtf((float)m));
    *full = t > dense || t * (float)m > 0.8f * (float)room ? mark : 0u;
  }
  if (!plan) return;
  bool own = lanes;
  uint32_t c = 0, best = L.sum[0];
#pragma unroll
  for (int k = 1; k < D; ++k)
    if (2u * L.sum[k] + 16u * S < best) {
      best = L.sum[k];
      c = (uint32_t)k;
    }
  if ((float)best > kClassCost * (float)L.sum[D] + 16.f * (float)S) own = true;
  float r[D], mc = (float)m;  // of class tid
  uint32_t cc = c;
#pragma unroll
  for (int k = 0; k < D; ++k) r[k] = (float)L.sum[k] / (float)S;
  if (own) {  // every class by its own samples
    if (tid < kPlanSamples) {
#pragma unroll
      for (int g = 0; g < D; ++g)
#pragma unroll
        for (int k = 0; k <= D; ++k) {
          const bool here = in && P.bk == (uint32_t)g;
          const uint32_t w = wave_scan_dpp(!here ? 0u : k < D ? P.est[k < D ? k : 0] : 1u);
          if (lane == kWave - 1) L.part[g * (D + 1) + k][wave] = w;
        }
    }
    sample_sums(L, D * (D + 1));
    if (tid < D) {
      const uint32_t* __restrict__ s = L.sum + tid * (D + 1);
      const float n = (float)max(s[D], 1u);
#pragma unroll
      for (int k = 0; k < D; ++k) r[k] = (float)s[k] / n;
      mc *= n / (float)S;
      cc = tid;
    }
  }
  // (a class of its own for the whole set has the others' cells too)
  const uint32_t all = own ? cells : D * cells;
  const uint32_t rows = own ? (uint32_t)D : 1u;  // rows of L.b: the classes, or the set's
  uint32_t* __restrict__ seen = sq[0];           // (the quantiles are read)
  static_assert(kSeen / 2 <= D * kQuantPad, "the counters take the quantiles' place");
  float least = 0.f;
  for (uint32_t finer = lanes ? kFinest : 0u; finer <= kFinest; ++finer) {
    if (tid < rows) L.reads[tid] = cell_shape<D>(mc, cc, all, r, finer, L.b[tid]);
    if (tid == 0) L.pairs = 0;
    for (uint32_t i = tid; i < kSeen / 2; i += kPlanThreads) seen[i] = 0;
    __syncthreads();
    if (tid < kPlanSamples) {
      uint32_t met = 0;  // samples in the cell already
      if (in) {
        const uint32_t g = own ? P.bk : c;
        const uint32_t i =
            (grid_cell<D>(L.b[own ? g : 0u], g, P.mid) + g * (kSeen / DDM_MAX_D + 1u)) & (kSeen - 1u);
        met = atomicAdd(&seen[i >> 1], i & 1u ? 0x10000u : 1u);
        met = i & 1u ? met >> 16 : met & 0xffffu;
      }
      const uint32_t sum = wave_scan_dpp(met);
      if (lane == kWave - 1) atomicAdd(&L.pairs, sum);
    }
    __syncthreads();
    const uint32_t pairs = L.pairs;
    float reads = 0.f;
    for (uint32_t g = 0; g < rows; ++g) reads += L.reads[g] / (float)rows;
    // a tile's share of the updates, or its cell's
    const float tile = (float)q / (float)m;
    const float cell = 2.f * (float)pairs / ((float)S * (float)S);
    const float cost = fmaxf(tile, cell) * reads;
    if ((finer == 0 || lanes || cost <= (finer < kFinest ? kFinerSlack : 1.f) * least) && tid < rows) {
      plan->cls = own ? kOwnClass : c;
#pragma unroll
      for (int s = 0; s < DDM_MAX_D; ++s) plan->b[cc][s] = L.b[tid][s];
    }
    least = finer == 0 ? cost : fminf(least, cost);
    if (finer == 0 && (pairs <= kCrowdedPairs || cell <= 2.f * tile)) return;
    __syncthreads();
  }
}

}  // namespace ddm
