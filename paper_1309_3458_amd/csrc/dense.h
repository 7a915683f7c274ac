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
// Measured on that workload, build + match: 20.7 -> 6.6 ms plain and 14.6 -> 6.3
// ms learned; 76,543 updates against 123,457 squares (247 pairs each): 0.45 ->
// 0.23 ms; 250,000 + 250,000 segments (d = 1, 100 pairs each): 0.46 -> 0.36 ms.
#pragma once

#include "traverse.h"

namespace ddm {

constexpr uint32_t kUnit = 1024;               // candidates of a unit
constexpr uint32_t kUnitBatches = kUnit / kWave;
// Units that one workgroup expands, and its wavefronts: long runs of writes where
// the lists are long; where most tiles have one unit, more and smaller workgroups
// (250,000 + 250,000 segments, lists of 300: 87 us with 4 units, 63 with one)
constexpr uint32_t kGroupLong = 4, kGroupShort = 1;
__host__ __device__ constexpr int expand_waves(uint32_t group) { return group > 1 ? 8 : 4; }
constexpr int kUnitWaves = 4;

struct DenseUnits {
  const uint64_t* toff = nullptr;   // first candidate of each tile, and the end
  const uint32_t* list = nullptr;   // candidate ids, ascending within a tile
  uint32_t* ubase = nullptr;        // first unit of each tile
  uint2* umap = nullptr;            // unit -> tile, index within the tile
  uint2* gmap = nullptr;            // group of units -> tile, its first unit
  uint32_t* ucount = nullptr;       // units, groups (zeroed beforehand)
  uint64_t* bits = nullptr;         // [tile][update][unit][batch]: hits
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

// units and groups of every tile (one thread per tile), in no particular order; a
// wavefront takes its places with one atomic for each of the two (8 us at 7800
// tiles with one a tile, 5 now)
__global__ __launch_bounds__(256) void dense_units_kernel(DenseUnits U, uint32_t tiles,
                                                          uint32_t group) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  const bool in = t < tiles;
  const uint32_t n = in ? (uint32_t)((U.toff[t + 1] - U.toff[t] + kUnit - 1) / kUnit) : 0u;
  const uint32_t g = (n + group - 1) / group;
  const uint32_t ni = wave_scan_dpp(n), gi = wave_scan_dpp(g);
  uint32_t b = 0, gb = 0;
  if (lane_id() == kWave - 1) {
    b = atomicAdd(U.ucount, ni);
    gb = atomicAdd(U.ucount + 1, gi);
  }
  b = readlane_u32(b, kWave - 1) + ni - n;
  gb = readlane_u32(gb, kWave - 1) + gi - g;
  if (!in) return;
  U.ubase[t] = b;
  for (uint32_t i = 0; i < n; ++i) U.umap[b + i] = make_uint2(t, i);
  for (uint32_t i = 0; i < g; ++i) U.gmap[gb + i] = make_uint2(t, i * group);
}

// a unit's candidates list[b0 .. b0 + len) and its tile's updates (lane: perm
// index's update j, none from nq on)
struct UnitSpan {
  uint64_t b0;
  uint32_t len, nq, j;
  uint32_t y, units;  // the unit's index in its tile, and the tile's units
};
template <int D>
__device__ __forceinline__ UnitSpan unit_span(const DenseUnits& U, const UpdSet& US, uint32_t u,
                                              uint32_t lane) {
  UnitSpan s;
  const uint2 w = U.umap[u];
  const uint32_t t = uniform_u32(w.x);
  s.y = uniform_u32(w.y);
  const uint64_t o = U.toff[t], a = o + (uint64_t)s.y * kUnit, e = U.toff[t + 1];
  s.units = uniform_u32((uint32_t)((e - o + kUnit - 1) / kUnit));
  s.b0 = a;
  s.len = uniform_u32((uint32_t)min<uint64_t>(e - a, kUnit));
  uint32_t k, qbeg;
  tile_span<D>(US, t, &k, &qbeg, &s.nq);
  s.j = lane < s.nq ? US.perm[qbeg + lane] : 0u;
  return s;
}

// Bound by the tests: 2D + 3 vector instructions for a candidate and 64
// updates.  The ids of the next batch but one and the records of the next are
// loaded while a batch is tested.  The masks are collected in LDS and written
// update by update, 8 batches (64 bytes) each; 16 at a time left LDS for four
// wavefronts a SIMD only (1.86 ms on the 16-hotspot workload, 1.68 with 8).
template <int D>
__global__ __launch_bounds__(kUnitWaves * kWave) void dense_test_kernel(
    DenseUnits U, UpdSet US, const float* __restrict__ rid, const float* __restrict__ ulo,
    const float* __restrict__ uhi, uint32_t m) {
  constexpr int R = 2 * D;
  __shared__ __align__(16) float s_cand[kUnitWaves][R * kWave];
  constexpr uint32_t kHold = 8;
  __shared__ uint64_t s_bits[kUnitWaves][kWave][kHold + 1];
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
  uint64_t* __restrict__ bits = U.bits + (size_t)(u - S.y) * kUnit + S.y * kUnitBatches;
  for (uint32_t b = 0; b < nb; ++b) {
    record(b + 1, idn, w);
    idn = id_of(b + 2);
    uint32_t mlo, mhi;
    test_masks<D>(ql, qh, S.nq, v, s_cand[wave], lane, min(S.len - b * kWave, (uint32_t)kWave),
                  true, &mlo, &mhi);
    s_bits[wave][lane][b % kHold] = (uint64_t)mhi << 32 | mlo;  // (0 from lane nq on)
    cnt += (uint32_t)__popc(mlo) + (uint32_t)__popc(mhi);
    wave_sync();  // the records are read before the next ones are put
    if (b % kHold == kHold - 1 || b + 1 == nb) {
      // 4 lanes to an update, two batches each
      const uint32_t h = b & ~(kHold - 1), c = 2 * (lane & 3u);
      for (uint32_t q = lane >> 2; q < S.nq; q += kWave / 4)
        if (h + c < nb)
          *reinterpret_cast<ulonglong2*>(bits + (size_t)q * S.units * kUnitBatches + h + c) =
              make_ulonglong2(s_bits[wave][q][c], s_bits[wave][q][c + 1]);
      wave_sync();
    }
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

// Keys from the masks.  A workgroup takes up to GROUP units of a tile, their ids
// in LDS, and its wavefronts the tile's updates in turn: an update's masks come
// with one load (a batch to a lane), its ids are packed into LDS, batch by batch,
// and written as keys to consecutive places of its segment, 64 at a time and in
// whole 128-byte lines but for the ends of the group.  Bound by the writes, 8
// bytes a pair.  On the 16-hotspot workload (1.8*10^9 pairs, 18 of 64 candidates
// are hits): 6.5 ms with stores straight from the masks (38 cycles each whatever
// they write); 8.6 with the updates inside the batches (64 open lines a
// wavefront); 4.6 with a unit to a wavefront, ids and masks in registers (runs of
// 290 pairs, lines written in two parts); 3.9 now, of which the packing alone
// takes 2.1.
template <int D, uint32_t GROUP>
__global__ __launch_bounds__(expand_waves(GROUP) * kWave) void dense_expand_kernel(
    DenseUnits U, UpdSet US, const uint64_t* __restrict__ off, uint64_t* __restrict__ out) {
  constexpr uint32_t kLine = 16;  // keys of a line
  constexpr uint32_t kPack = kUnit + 2 * kLine;
  constexpr int kExpandWaves = expand_waves(GROUP);
  constexpr uint32_t kThreads = kExpandWaves * kWave, kIds = GROUP * kUnit;
  __shared__ uint32_t s_ids[kIds];
  __shared__ uint32_t s_pack[kExpandWaves][kPack + 1];  // and one for the lanes without a hit
  const uint32_t gi = blockIdx.x;
  if (gi >= uniform_u32(U.ucount[1])) return;
  const uint32_t lane = lane_id(), wave = uniform_u32(threadIdx.x / kWave);
  uint32_t* __restrict__ pack = s_pack[wave];
  const uint2 gw = U.gmap[gi];
  const uint32_t t = uniform_u32(gw.x), y0 = uniform_u32(gw.y);
  const uint64_t tb = U.toff[t], te = U.toff[t + 1];
  const uint32_t u0 = uniform_u32(U.ubase[t]);
  const uint32_t row = uniform_u32((uint32_t)((te - tb + kUnit - 1) / kUnit)) * kUnitBatches;
  const uint64_t b0 = tb + (uint64_t)y0 * kUnit;
  const uint32_t len = uniform_u32((uint32_t)min<uint64_t>(te - b0, kIds));
  uint32_t v[kIds / kThreads];
#pragma unroll
  for (uint32_t r = 0; r < kIds / kThreads; ++r) {
    const uint32_t i = r * kThreads + threadIdx.x;
    v[r] = i < len ? U.list[b0 + i] : 0u;
  }
  uint32_t k, qbeg, nq;
  tile_span<D>(US, t, &k, &qbeg, &nq);
  const uint32_t j = lane < nq ? US.perm[qbeg + lane] : 0u;
  // lane: its update's first place of the group
  const uint64_t base = lane < nq ? off[j] + U.ucnt[(size_t)(u0 + y0) * kWave + lane] : 0ull;
  const uint32_t nb = (len + kWave - 1) / kWave;
  // one load brings the masks of kRows updates, a batch to a lane
  constexpr uint32_t kRow = GROUP * kUnitBatches, kRows = kWave / kRow;
  static_assert(kRows * kRow == kWave, "whole rows");
  const uint64_t* __restrict__ masks =
      U.bits + (size_t)u0 * kUnit + y0 * kUnitBatches + lane % kRow;
  auto masks_of = [&](uint32_t first) {
    const uint32_t q = first + lane / kRow;
    return q < nq && lane % kRow < nb ? masks[(size_t)q * row] : 0ull;
  };
  uint64_t next = masks_of(wave * kRows);
#pragma unroll
  for (uint32_t r = 0; r < kIds / kThreads; ++r) s_ids[r * kThreads + threadIdx.x] = v[r];
  __syncthreads();
  uint64_t mine = 0, some = 0;
  for (uint32_t i = 0, q = wave * kRows; q < nq; ++i) {
    const uint32_t r = i % kRows;
    if (r == 0) {
      mine = next;
      next = masks_of(q + kExpandWaves * kRows);
      some = ballot(mine != 0);
    }
    const uint32_t here = q, r0 = r * kRow;
    q += r == kRows - 1 ? (kExpandWaves - 1) * kRows + 1 : 1;
    if (!((some >> r0) & (~0ull >> (kWave - kRow)))) continue;
    const uint64_t at = readlane_u64(base, here);
    const uint32_t who = readlane_u32(j, here);
    // from the start of the line the run begins in: pack[i] goes to dst[i]
    uint32_t skip = (uint32_t)(((uintptr_t)(out + at) >> 3) & (kLine - 1));
    uint64_t* __restrict__ dst = out + at - skip;
    uint32_t n = skip;
#pragma unroll
    for (uint32_t y = 0; y < GROUP; ++y) {
      const bool last = (y + 1) * kUnitBatches >= nb;
#pragma unroll
      for (uint32_t c = 0; c < kUnitBatches; c += 4) {
        if (y * kUnitBatches + c < nb) {
#pragma unroll
          for (uint32_t b = y * kUnitBatches + c; b < y * kUnitBatches + c + 4; ++b) {
            const uint64_t m = readlane_u64(mine, r0 + b);
            const uint32_t to = mask_rank_from(m, n);
            pack[lane_of(m) ? to : kPack] = s_ids[b * kWave + lane];
            n += (uint32_t)__popcll(m);
          }
        }
      }
      wave_sync();
      // to the end of the run, or to the last line that is full
      const uint32_t end = last ? n : n & ~(kLine - 1);
      for (uint32_t i0 = 0; i0 < end; i0 += 4 * kWave) {
        uint32_t p[4];  // (their reads are in flight together)
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) p[r] = pack[min(i0 + r * kWave + lane, kPack)];
        uint64_t* __restrict__ to = dst + i0;
        const uint32_t room = end - i0;
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
          const uint32_t i = r * kWave + lane;
          if (i < room && (r > 0 || i0 + lane >= skip)) to[i] = (uint64_t)who << 32 | p[r];
        }
      }
      if (last) break;
      if (end) {  // what is left moves to the front
        if (end + lane < n) {
          const uint32_t w = pack[end + lane];
          wave_sync();
          pack[lane] = w;
        }
        n -= end;
        dst += end;
        skip = 0;
      }
      wave_sync();
    }
    wave_sync();
  }
}

}  // namespace ddm
