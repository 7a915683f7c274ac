// Matching of dense sets: the pairs leave the traversal already in
// subscription order, so that no segment is sorted.
//
// A tile's updates are neighbours, so their candidates (the subscriptions that
// meet the tile's enclosing box) are few compared with the pairs: on the
// 16-hotspot workload about 12,000 of them against 250,000 pairs of a tile.
// Each tile's candidate ids are listed and the lists sorted (a fifteenth of
// the keys that the pairs have); the updates are then tested against the
// sorted list, 64 candidates at a time, and every update's hits come out in
// id order.  The work unit is a tile and up to kUnit candidates of its list,
// so that a long list spreads over many wavefronts.  A unit keeps the hit
// masks it computes (one bit per test); once the counts are summed and
// scanned, a second kernel expands the masks into keys at their final places,
// the only time the pairs move.
// Measured on that workload, build + match: 20.7 -> 8.3 ms plain and 14.4 -> 7.7
// ms learned; 76,543 updates against 123,457 squares (247 pairs each): 0.45 ->
// 0.28 ms; 250,000 + 250,000 segments (d = 1, 200 pairs each): 0.45 -> 0.41 ms.
#pragma once

#include "traverse.h"

namespace ddm {

constexpr uint32_t kUnit = 1024;               // candidates of a unit
constexpr uint32_t kUnitBatches = kUnit / kWave;
constexpr int kUnitWaves = 4;

struct DenseUnits {
  const uint64_t* toff = nullptr;   // first candidate of each tile, and the end
  const uint32_t* list = nullptr;   // candidate ids, ascending within a tile
  uint32_t* ubase = nullptr;        // first unit of each tile
  uint2* umap = nullptr;            // unit -> tile, index within the tile
  uint32_t* ucount = nullptr;       // units (zeroed beforehand)
  uint2* bits = nullptr;            // [unit][batch][lane]: hits of the lane's update
  uint32_t* ucnt = nullptr;         // [unit][lane]: hits, then those of the units before
};

// the updates of tile `item` (uniform): class k, first perm index, count
template <int D>
__device__ __forceinline__ void tile_span(const UpdSet& US, uint32_t item, uint32_t* k_out,
                                          uint32_t* qbeg_out, uint32_t* nq_out) {
  uint32_t k = 0, qbeg = 0, nq = 0;
  if (US.tstart) {
    k = US.tclass[item];
    qbeg = US.tstart[item];
    nq = US.tstart[item + 1] - qbeg;
  } else {
    uint32_t t = item;
#pragma unroll
    for (int g = 0; g < D; ++g) {
      const uint32_t c = uniform_u32(US.gcount[g]);
      const uint32_t nt = (c + US.qpt - 1) / US.qpt;
      if (nq == 0 && t < nt) {
        k = (uint32_t)g;
        qbeg = US.gstart[g] + t * US.qpt;
        nq = min(US.qpt, c - t * US.qpt);
      }
      t -= min(t, nt);
    }
  }
  *k_out = uniform_u32(k);
  *qbeg_out = uniform_u32(qbeg);
  *nq_out = uniform_u32(nq);
}

// the enclosing box of every tile (dimension-major, like the updates): lists
// sized by the predictor take its estimate for the box (one wavefront per tile)
template <int D>
__global__ __launch_bounds__(kUnitWaves * kWave) void tile_boxes_kernel(
    UpdSet US, const float* __restrict__ ulo, const float* __restrict__ uhi, uint32_t m,
    uint32_t tiles, float* __restrict__ blo, float* __restrict__ bhi) {
  const uint32_t lane = lane_id();
  const uint32_t t = uniform_u32(blockIdx.x * kUnitWaves + threadIdx.x / kWave);
  if (t >= tiles) return;
  uint32_t k, qbeg, nq;
  tile_span<D>(US, t, &k, &qbeg, &nq);
  const uint32_t j = lane < nq ? US.perm[qbeg + lane] : US.perm[qbeg];
#pragma unroll
  for (int s = 0; s < D; ++s) {
    const float a = wave_min(ulo[(size_t)s * m + j]), b = wave_max(uhi[(size_t)s * m + j]);
    if (lane == 0) {
      blo[(size_t)s * tiles + t] = a;
      bhi[(size_t)s * tiles + t] = b;
    }
  }
}

// a tile's list gets half as much again as the predictor says, and 64 more
// (tiles past the last one, of a class that ended early: none)
__global__ __launch_bounds__(256) void tile_room_kernel(uint32_t* __restrict__ cap, uint32_t tiles,
                                                        uint32_t n) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < tiles) cap[t] = min(cap[t] + cap[t] / 2u + 64u, n);
}

// the part of each list that fitted; *over counts the tiles that had more
__global__ __launch_bounds__(256) void tile_clip_kernel(const uint32_t* __restrict__ tcand,
                                                        const uint32_t* __restrict__ cap,
                                                        uint32_t tiles, uint32_t* __restrict__ len,
                                                        uint64_t* __restrict__ over) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = t < tiles;
  const uint32_t c = in ? tcand[t] : 0u, r = in ? cap[t] : 0u;
  if (in) len[t] = min(c, r);
  const uint64_t bad = ballot(c > r);
  if (bad && lane_id() == 0) atomicAdd((unsigned long long*)over, (unsigned long long)__popcll(bad));
}

// units of every tile (one thread per tile), in no particular order
__global__ __launch_bounds__(256) void dense_units_kernel(DenseUnits U, uint32_t tiles) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= tiles) return;
  const uint32_t n = (uint32_t)((U.toff[t + 1] - U.toff[t] + kUnit - 1) / kUnit);
  const uint32_t b = n ? atomicAdd(U.ucount, n) : 0u;
  U.ubase[t] = b;
  for (uint32_t i = 0; i < n; ++i) U.umap[b + i] = make_uint2(t, i);
}

// a unit's candidates list[b0 .. b0 + len) and its tile's updates (lane: perm
// index's update j, none from nq on)
struct UnitSpan {
  uint64_t b0;
  uint32_t len, nq, j;
};
template <int D>
__device__ __forceinline__ UnitSpan unit_span(const DenseUnits& U, const UpdSet& US, uint32_t u,
                                              uint32_t lane) {
  UnitSpan s;
  const uint2 w = U.umap[u];
  const uint32_t t = uniform_u32(w.x);
  const uint64_t a = U.toff[t] + (uint64_t)uniform_u32(w.y) * kUnit, e = U.toff[t + 1];
  s.b0 = a;
  s.len = uniform_u32((uint32_t)min<uint64_t>(e - a, kUnit));
  uint32_t k, qbeg;
  tile_span<D>(US, t, &k, &qbeg, &s.nq);
  s.j = lane < s.nq ? US.perm[qbeg + lane] : 0u;
  return s;
}

// Bound by the tests: 2D + 3 vector instructions for a candidate and 64
// updates.  The ids of the next batch but one and the records of the next are
// loaded while a batch is tested.
template <int D>
__global__ __launch_bounds__(kUnitWaves * kWave) void dense_test_kernel(
    DenseUnits U, UpdSet US, const float* __restrict__ rid, const float* __restrict__ ulo,
    const float* __restrict__ uhi, uint32_t m) {
  constexpr int R = 2 * D;
  __shared__ __align__(16) float s_cand[kUnitWaves][R * kWave];
  const uint32_t lane = lane_id(), wave = threadIdx.x / kWave;
  const uint32_t u = uniform_u32(blockIdx.x * kUnitWaves + wave);
  if (u >= uniform_u32(*U.ucount)) return;
  const UnitSpan S = unit_span<D>(U, US, u, lane);
  float ql[D], qh[D];
#pragma unroll
  for (int s = 0; s < D; ++s) {
    ql[s] = lane < S.nq ? ulo[(size_t)s * m + S.j] : INFINITY;
    qh[s] = lane < S.nq ? uhi[(size_t)s * m + S.j] : -INFINITY;
  }
  const uint32_t* __restrict__ ids = U.list + S.b0;
  const uint32_t nb = (S.len + kWave - 1) / kWave;
  auto record = [&](uint32_t b, uint32_t id, float (&v)[R]) {
    if (b * kWave + lane < S.len) {
      load_rec<D>(rid + (size_t)id * R, v);
    } else {
#pragma unroll
      for (int s = 0; s < D; ++s) {
        v[2 * s] = INFINITY;
        v[2 * s + 1] = -INFINITY;
      }
    }
  };
  auto id_of = [&](uint32_t b) { return b * kWave + lane < S.len ? ids[b * kWave + lane] : 0u; };
  float v[R], w[R];
  record(0, id_of(0), v);
  uint32_t idn = id_of(1), cnt = 0;
  uint2* __restrict__ bits = U.bits + (size_t)u * kUnit;
  for (uint32_t b = 0; b < nb; ++b) {
    record(b + 1, idn, w);
    idn = id_of(b + 2);
    uint32_t mlo, mhi;
    test_masks<D>(ql, qh, S.nq, v, s_cand[wave], lane, min(S.len - b * kWave, (uint32_t)kWave),
                  true, &mlo, &mhi);
    bits[b * kWave + lane] = make_uint2(mlo, mhi);  // (0 from lane nq on)
    cnt += (uint32_t)__popc(mlo) + (uint32_t)__popc(mhi);
    wave_sync();  // the records are read before the next ones are put
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = w[r];
  }
  U.ucnt[(size_t)u * kWave + lane] = cnt;
}

// per tile: the units' counts of every update to the counts of the units
// before, and the updates' totals (one wavefront per tile)
template <int D>
__global__ __launch_bounds__(kUnitWaves * kWave) void dense_sum_kernel(DenseUnits U, UpdSet US,
                                                                      uint32_t tiles,
                                                                      uint32_t* __restrict__ cnt) {
  const uint32_t lane = lane_id();
  const uint32_t t = uniform_u32(blockIdx.x * kUnitWaves + threadIdx.x / kWave);
  if (t >= tiles) return;
  uint32_t k, qbeg, nq;
  tile_span<D>(US, t, &k, &qbeg, &nq);
  const uint32_t n = (uint32_t)((U.toff[t + 1] - U.toff[t] + kUnit - 1) / kUnit);
  uint32_t* __restrict__ c = U.ucnt + (size_t)U.ubase[t] * kWave + lane;
  uint32_t run = 0;
  for (uint32_t i = 0; i < n; i += 4) {
    uint32_t v[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) v[q] = i + q < n ? c[(size_t)(i + q) * kWave] : 0u;
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      if (i + q < n) c[(size_t)(i + q) * kWave] = run;
      run += v[q];
    }
  }
  if (lane < nq) cnt[US.perm[qbeg + lane]] = run;
}

// Keys from the masks.  The unit's ids and masks are loaded into registers; then
// one update after the other packs the ids it meets into LDS, batch by batch,
// and writes them as keys to consecutive places of its segment, 64 at a time and
// in whole 128-byte lines but for the ends.  Stores straight from the masks (18
// of 64 lanes active on the 16-hotspot workload) took 38 cycles each whatever
// they wrote, 6.5 ms for its 1.8*10^9 pairs; with the updates inside the batches
// each wavefront also had 64 partly written lines open, 8.6 ms; this form
// 4.6 ms.  Bound by the writes, 8 bytes a pair.
template <int D>
__global__ __launch_bounds__(kUnitWaves * kWave) void dense_expand_kernel(
    DenseUnits U, UpdSet US, const uint64_t* __restrict__ off, uint64_t* __restrict__ out) {
  __shared__ uint32_t s_ids[kUnitWaves][kUnit];
  uint32_t* __restrict__ pack = s_ids[threadIdx.x / kWave];
  const uint32_t lane = lane_id();
  const uint32_t u = uniform_u32(blockIdx.x * kUnitWaves + threadIdx.x / kWave);
  if (u >= uniform_u32(*U.ucount)) return;
  const UnitSpan S = unit_span<D>(U, US, u, lane);
  const uint64_t base = lane < S.nq ? off[S.j] + U.ucnt[(size_t)u * kWave + lane] : 0ull;
  const uint32_t* __restrict__ ids = U.list + S.b0;
  const uint2* __restrict__ bits = U.bits + (size_t)u * kUnit;
  const uint32_t nb = (S.len + kWave - 1) / kWave;
  uint32_t id[kUnitBatches];
  uint2 mk[kUnitBatches];
  uint32_t any = 0;
#pragma unroll
  for (uint32_t b = 0; b < kUnitBatches; ++b) {
    id[b] = 0;
    mk[b] = make_uint2(0u, 0u);
    if (b < nb) {  // (the last batch: no mask has a bit past the unit's end)
      id[b] = ids[min(b * kWave + lane, S.len - 1u)];
      mk[b] = bits[b * kWave + lane];
    }
  }
#pragma unroll
  for (uint32_t b = 0; b < kUnitBatches; ++b) any |= mk[b].x | mk[b].y;
  uint64_t some = ballot(any != 0);
  while (some) {
    const uint32_t q = (uint32_t)__builtin_ctzll(some);
    some &= some - 1;
    const uint64_t at = readlane_u64(base, q);
    const uint64_t jq = (uint64_t)readlane_u32(S.j, q) << 32;
    uint32_t n = 0;
#pragma unroll
    for (uint32_t b = 0; b < kUnitBatches; ++b) {
      if (b < nb) {
        const uint64_t m = (uint64_t)readlane_u32(mk[b].y, q) << 32 | readlane_u32(mk[b].x, q);
        if (lane_of(m)) pack[n + mask_rank(m)] = id[b];
        n += (uint32_t)__popcll(m);
      }
    }
    wave_sync();
    // from the start of the line the run begins in
    const uint32_t skip = (uint32_t)(((uintptr_t)(out + at) >> 3) & 15u);
    uint64_t* __restrict__ dst = out + at - skip;
    for (uint32_t i = lane; i < n + skip; i += kWave)
      if (i >= skip) dst[i] = jq | pack[i - skip];
    wave_sync();
  }
}

}  // namespace ddm
