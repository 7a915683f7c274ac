// Device-side pieces shared by the single-instance and batched matchers:
// record/query loads, wavefront helpers, the update-set and output-segment
// descriptors, and the body of the tile traversal.
#pragma once

#include "ddm_internal.h"

#include <algorithm>
#include <cmath>

namespace ddm {

// --------------------------------------------------------------------------
// helpers
// --------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void load_rec(const float* __restrict__ p, float (&v)[2 * D]) {
  if constexpr (D == 1) {
    const float2 a = *reinterpret_cast<const float2*>(p);
    v[0] = a.x; v[1] = a.y;
  } else if constexpr (D == 2) {
    const float4 a = *reinterpret_cast<const float4*>(p);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  } else if constexpr (D == 3) {
    const float2 a = reinterpret_cast<const float2*>(p)[0];
    const float2 b = reinterpret_cast<const float2*>(p)[1];
    const float2 c = reinterpret_cast<const float2*>(p)[2];
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y; v[4] = c.x; v[5] = c.y;
  } else {
    const float4 a = reinterpret_cast<const float4*>(p)[0];
    const float4 b = reinterpret_cast<const float4*>(p)[1];
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
}

template <int D>
__device__ __forceinline__ void store_rec(float* __restrict__ p, const float (&v)[2 * D]) {
  if constexpr (D == 2 || D == 4) {
#pragma unroll
    for (int q = 0; q < D / 2; ++q)
      reinterpret_cast<float4*>(p)[q] =
          make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  } else {
#pragma unroll
    for (int q = 0; q < D; ++q)
      reinterpret_cast<float2*>(p)[q] = make_float2(v[2 * q], v[2 * q + 1]);
  }
}

// Query j's bounds in record order: probe dimension k first, then the other
// dimensions ascending (slot s >= 1 holds dimension s-1 or s).
template <int D>
__device__ __forceinline__ void load_query(const float* __restrict__ ulo,
                                           const float* __restrict__ uhi, uint32_t m,
                                           uint32_t j, uint32_t k, float (&ql)[D],
                                           float (&qh)[D]) {
  ql[0] = ulo[(size_t)k * m + j];
  qh[0] = uhi[(size_t)k * m + j];
#pragma unroll
  for (int s = 1; s < D; ++s) {
    const uint32_t kk = (uint32_t)(s - 1) + (((uint32_t)(s - 1) >= k) ? 1u : 0u);
    ql[s] = ulo[(size_t)kk * m + j];
    qh[s] = uhi[(size_t)kk * m + j];
  }
}

// closed overlap of a record (2D floats) with query bounds, all dimensions
template <int D>
__device__ __forceinline__ bool overlaps(const float (&v)[2 * D], const float (&ql)[D],
                                         const float (&qh)[D]) {
  bool ok = true;
#pragma unroll
  for (int s = 0; s < D; ++s) ok = ok && (v[2 * s] <= qh[s]) && (ql[s] <= v[2 * s + 1]);
  return ok;
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  return wave_fold_dpp(v, [](uint32_t a, uint32_t b) { return min(a, b); });
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  return wave_fold_dpp(v, [](uint32_t a, uint32_t b) { return max(a, b); });
}

__device__ __forceinline__ uint32_t readlane_u32(uint32_t v, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}
__device__ __forceinline__ float readlane_f32(float v, uint32_t lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), (int)lane));
}
// v with lane `lane` replaced by x (both uniform); the compiler has the
// intrinsic but no builtin for it
extern "C" __device__ int ddm_writelane(int x, int lane, int v) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ uint32_t writelane_u32(uint32_t v, uint32_t x, uint32_t lane) {
  return (uint32_t)ddm_writelane((int)x, (int)lane, (int)v);
}
// 2 acc + (this lane's bit of m): one add with the mask as the carries
__device__ __forceinline__ uint32_t shift_in(uint32_t acc, uint64_t m) {
  uint32_t r;
  asm("v_addc_co_u32_e64 %0, vcc, %1, %1, %2" : "=v"(r) : "v"(acc), "s"(m) : "vcc");
  return r;
}
// whether this lane's bit of the (uniform) mask is set
__device__ __forceinline__ bool lane_of(uint64_t m) {
  return __builtin_amdgcn_inverse_ballot_w64(m);
}

__device__ __forceinline__ uint64_t readlane_u64(uint64_t v, uint32_t lane) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, (int)lane);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), (int)lane);
  return ((uint64_t)hi << 32) | lo;
}

// Which updates a traversal processes: group g (probe dimension g) holds
// gcount[g] updates at perm[gstart[g] ...].
struct UpdSet {
  const uint32_t* perm;
  const uint32_t* gstart;
  const uint32_t* gcount;
  uint32_t total;     // upper bound of sum(gcount), for the launch size
  uint32_t qpt = 64;  // updates per wavefront in the tile traversal
  // optional: per update j, pb[2j] <= the first and pb[2j+1] >= the last
  // position of its candidate range in its probe tree (bounds from the
  // probe's quantile searches); tiles then skip their own searches
  const uint32_t* pb = nullptr;
  // optional tile list (replaces the tiles of qpt updates): tile t holds
  // perm[tstart[t] .. tstart[t+1]) (at most 64 updates of one class), belongs
  // to class tclass[t], and there are *ntiles tiles
  const uint32_t* tstart = nullptr;
  const uint32_t* tclass = nullptr;
  const uint64_t* ntiles = nullptr;
  bool refill = false;  // the updates that overflowed their slots (names the kernel's record)
};

// Where a traversal writes.  COUNT (fill == false): cnt[j] = hits of j.
// FILL: hit r of update j goes to out[base[j] + r] if that is below the
// segment end: base[j+1] (final offsets, cap == nullptr) or
// min(base[j] + cap[j], limit) (slots of the single-pass form); with cnt
// non-null the total number of hits (written or not) is stored in cnt[j].
// COUNT with a stash (skey non-null, tile traversal only): every hit is also
// appended, with its rank among its update's hits, to chunks of kStashChunk
// entries.  Tile t owns chunks kStashStatic*t .. +kStashStatic-1 (no atomic
// for tiles with few hits); further chunks come from the slice
// t % kStashSlices of the counted chunks, at least kStashGrab at a time
// (the tile keeps the surplus for its next hits): slice s spans sslice
// chunks from sfirst + s*sslice and snext[s] is its next free chunk
// (separate counters, so that tiles do not queue on one address).  snext[kStashSlices] becomes
// non-zero once a slice is used up (the stash is then incomplete and the
// counts alone are valid).  sused[c] = entries written in chunk c; every
// tile writes it for each of its static chunks.
constexpr uint32_t kStashChunk = 64;
constexpr uint32_t kStashStatic = 2;
constexpr uint32_t kStashSlices = 256;
// snext[kStashSlices]: 1 overflow, 2 (set before the count) a dense set
constexpr uint32_t kStashDense = 2;
// (a slice has a line of its own, sum and maximum: with the slices packed, the
// atomics of 7800 tiles queued on six lines, 46 us for a traversal that takes 17)
constexpr uint32_t kListSlices = 64, kListPad = 16;
constexpr uint32_t kStashGrab = 4;  // at least this many counted chunks per request
// at most 2^28 stashed hits (4 GiB of stash); larger results overflow it and
// take the fill traversal
constexpr uint64_t kStashMaxEntries = 1ull << 28;
// the stash has room for a caller's capacity up to this many hits per update: what
// has more is matched from candidate lists, or filled by a second traversal (with a
// batch, which has no lists, no stash beyond it: 2 hits per update gain, 18 lose)
constexpr uint64_t kStashMaxPerUpdate = 8;

struct SegOut {
  const uint64_t* base;
  const uint32_t* cap;
  uint64_t limit;
  uint32_t* cnt;
  uint64_t* out;
  // FILL, optional: the subscription id of each hit (4 bytes) at the same
  // place in this array instead of the key in out (the segment sort then
  // forms the keys as it writes them)
  uint32_t* ids = nullptr;
  uint64_t* skey = nullptr;
  uint32_t* srank = nullptr;
  uint32_t* sused = nullptr;
  uint32_t* snext = nullptr;
  uint32_t* sowner = nullptr;  // optional: tile of every counted chunk a tile takes
  uint32_t sfirst = 0;
  uint32_t sslice = 0;
  // LIST, and the stash form of a dense set (tcand optional in LIST): the number
  // of candidates of each tile, their sums and maxima over the tiles t with t %
  // kListSlices alike; LIST with ids: the ids of tile t's candidates, as far as
  // they fit, to ids[base[t] .. base[t + 1])
  uint32_t* tcand = nullptr;
  uint64_t* tsum = nullptr;
};

__device__ __forceinline__ bool upd_index(const UpdSet& U, uint32_t t, uint32_t d,
                                          uint32_t* idx, uint32_t* grp = nullptr) {
  uint32_t acc = 0;
  for (uint32_t g = 0; g < d; ++g) {
    const uint32_t c = U.gcount[g];
    if (t < acc + c) {
      *idx = U.gstart[g] + (t - acc);
      if (grp) *grp = g;
      return true;
    }
    acc += c;
  }
  return false;
}

__device__ __forceinline__ void seg_bounds(const SegOut& O, uint32_t j, uint64_t* b,
                                           uint64_t* e) {
  *b = O.base[j];
  if (O.cap) {
    const uint64_t e0 = *b + O.cap[j];
    *e = e0 < O.limit ? e0 : (O.limit > *b ? O.limit : *b);
  } else {
    *e = O.base[j + 1];
  }
}

// --------------------------------------------------------------------------
// 3/5b. one wavefront per tile of up to 64 updates (same probe dimension k,
// consecutive in the cell order).
//
// The tile's candidates in tree k are confined to positions
// [Pbeg, Pend] = [min plo, max phi] of its updates.  The wave walks that
// range block by block (64 positions; the tree's maxupper of position 64c and
// of the height-5 subtree at 64c+32, i.e. Algorithm 4's pruning test cut at
// height 5): 64 lanes read 64 block maxima at once and a ballot keeps the
// blocks whose maxupper reaches the tile's smallest q.lower.  A kept block is
// read one position per lane; positions meeting the tile's enclosing box in
// every dimension are compacted into an LDS ring with a ballot and a prefix
// popcount.  Each time 64 candidates are pending, lane l takes candidate l
// and the wave tests the tile's updates one after the other against the 64
// candidates (Algorithm 1, closed, every dimension): the ballot of the test
// is the update's hits among them, and a prefix popcount places the hits
// contiguously in the update's own segment.
// --------------------------------------------------------------------------
// d > 1: a tile whose range spans at least kStripRange positions takes the
// blocks of the strips it touches instead (tree_dev.h), testing 64 block
// boxes at once.  Shorter ranges hold fewer blocks than the 32 of a strip.
constexpr uint32_t kChunkPosLog = 11;  // positions of a strip
constexpr uint32_t kStripRange = 1024;
// Consecutive updates may lie far apart, where a line of cells ends or a cluster
// does, and the tile's box then holds all that lies between them: one such tile can
// take longer than all others together (500,000 squares in 16 clusters, 5857
// candidates in one tile where 250 are usual: count 337 us, 85 now).  Where more
// than kManyBlocks of 64 blocks meet the box, those that meet no update's own are
// dropped; a tile whose blocks stay is dense, and does not try again.  (With 8 in
// place of 24 at d = 4: 200,000 + 200,000 boxes, 50 hits each, match 352 us, 390.)
constexpr int kManyBlocks = 8, kManyBlocks4 = 24;  // d <= 3, d = 4
constexpr int kTileWaves = 4;
constexpr int kRing = 128;

// One tile of the traversal: updates perm[qbeg .. qbeg + nq) (global indices;
// qoff is subtracted to index the instance's coordinates), probe dimension k
// of tree set T.  LDS per wavefront: s_cand [kRing][2D] floats (records), s_cid
// [kRing].
//
// Candidates are tested 64 at a time (a flush), in one of two forms, whichever
// takes fewer vector instructions; both leave in lane u the mask of the
// candidates that update u meets:
//   by candidate: the update's bounds sit in its lane, every candidate is
//     compared with all updates at once (its first dimension from the lane
//     that holds it, the others broadcast from LDS), and the result is shifted
//     into each lane's mask with one add-with-carry: 2 + 2D + 1 instructions
//     for a candidate, whatever the number of updates;
//   by update: every lane holds a candidate, the update's bounds come from its
//     lane, and its mask is written to that lane: 4D + 2 instructions for an
//     update, whatever the number of candidates.
// Reading each update's bounds from LDS, with a ballot, a lane extract and a
// count per update, took about 31 instructions for an update; a window search
// per candidate over the updates sorted in a second dimension took fewer only
// where cells were wide (10^6 boxes, d = 3, count with strips and cells alike:
// 217 us with it, 177 us this way).

// Tests 64 candidates (lane l holds record v of candidate l; past c they are
// empty) against the updates of the lanes (bounds ql, qh; lanes from nq on hold
// none): *mlo and *mhi receive the mask of the candidates that the lane's update
// meets.  cd: 64 records of LDS; lanes with `put` write theirs there first if
// they are read.
template <int D>
__device__ __forceinline__ void test_masks(const float (&ql)[D], const float (&qh)[D], uint32_t nq,
                                           const float (&v)[2 * D], float* __restrict__ cd,
                                           uint32_t lane, uint32_t c, bool put, uint32_t* mlo_out,
                                           uint32_t* mhi_out) {
  constexpr int R = 2 * D;
  uint32_t mlo = 0, mhi = 0;
  const uint32_t groups = (c + 15u) / 16u;
  if (groups * 16u * (2u * D + 3u) < nq * (4u * D + 2u)) {
    if (D > 1) {
      if (put) store_rec<D>(cd + lane * R, v);
      wave_sync();
    }
    for (uint32_t g = 0; g < groups; ++g) {
      const float* __restrict__ cg = cd + 16u * g * R;
      uint32_t acc = 0;
#pragma unroll
      for (int i = 15; i >= 0; --i) {
        const uint32_t ln = 16u * g + (uint32_t)i;
        uint64_t m = ballot(readlane_f32(v[0], ln) <= qh[0]);
        m &= ballot(ql[0] <= readlane_f32(v[1], ln));
#pragma unroll
        for (int s = 1; s < D; ++s) {
          const float2 b = *reinterpret_cast<const float2*>(cg + i * R + 2 * s);
          m &= ballot(b.x <= qh[s]);
          m &= ballot(ql[s] <= b.y);
        }
        acc = shift_in(acc, m);
      }
      if (g < 2) mlo |= acc << (16u * g);
      else mhi |= acc << (16u * (g - 2u));
    }
  } else {
    for (uint32_t u0 = 0; u0 < nq; u0 += 4) {
#pragma unroll
      for (uint32_t q = 0; q < 4; ++q) {
        const uint32_t u = u0 + q;  // below 64; lanes from nq on meet nothing
        uint64_t m = ~0ull;
#pragma unroll
        for (int s = 0; s < D; ++s) {
          m &= ballot(v[2 * s] <= readlane_f32(qh[s], u));
          m &= ballot(readlane_f32(ql[s], u) <= v[2 * s + 1]);
        }
        mlo = writelane_u32(mlo, (uint32_t)m, u);
        mhi = writelane_u32(mhi, (uint32_t)(m >> 32), u);
      }
    }
  }
  *mlo_out = mlo;
  *mhi_out = mhi;
}

// whether a block's box b meets that of any of the tile's nq updates
template <int D>
__device__ __forceinline__ bool meets_any(const float (&b)[2 * D], const float (&ql)[D],
                                          const float (&qh)[D], uint32_t nq) {
  bool any = false;
  for (uint32_t u = 0; u < nq; ++u) {
    bool ok = true;
#pragma unroll
    for (int s = 0; s < D; ++s)
      ok = ok & (b[2 * s] <= readlane_f32(qh[s], u)) & (readlane_f32(ql[s], u) <= b[2 * s + 1]);
    any = any | ok;
  }
  return any;
}

enum TileMode {
  kTileCount,  // counts
  kTileFill,   // hits into the updates' segments or slots, counts if asked
  kTileStash,  // counts and kept hits; a set marked dense: as kTileList
  kTileList    // the tile's candidates: their number, or their ids
};

template <int D, TileMode MODE>
__device__ __forceinline__ void tile_body(const TreeDev& T, const float* __restrict__ ulo,
                                          const float* __restrict__ uhi, uint32_t m,
                                          const uint32_t* __restrict__ perm, uint32_t qoff,
                                          uint32_t k, uint32_t qbeg, uint32_t nq, const SegOut& O,
                                          float* __restrict__ s_cand, uint32_t* __restrict__ s_cid,
                                          uint32_t lane, uint32_t tile_id = 0,
                                          const uint32_t* __restrict__ pb = nullptr) {
  constexpr int R = 2 * D;
  constexpr bool FILL = MODE == kTileFill, STASH = MODE == kTileStash;
  nq = uniform_u32(nq);
  const uint32_t sflag = STASH ? uniform_u32(O.snext[kStashSlices]) : 0u;
  const bool listing = MODE == kTileList || (STASH && (sflag & kStashDense));
  const bool qv = lane < nq;
  const uint32_t gj = qv ? perm[qbeg + lane] : 0u;  // global update index
  const uint32_t j = gj - qoff;                      // index within the instance
  float ql[D], qh[D];
  if (qv) {
    load_query<D>(ulo, uhi, m, j, k, ql, qh);
  } else {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      ql[s] = INFINITY;
      qh[s] = -INFINITY;
    }
  }
  float elo[D], ehi[D];
#pragma unroll
  for (int s = 0; s < D; ++s) {
    elo[s] = wave_min(ql[s]);
    ehi[s] = wave_max(qh[s]);
  }
  // candidate positions of the tile in tree k: lower bound in
  // [t, Ehi] with t <= Elo - maxlen (see the probe kernels).  With per-update
  // bounds from the probe (a superset of each update's range; every
  // position scanned is still tested exactly), the tile's range is their
  // union; otherwise two-level searches over the sorted lower bounds.
  uint32_t Pbeg, Pend;
  if (pb) {
    uint32_t b0 = 0xffffffffu, e0 = 0u;
    if (qv) {
      const uint2 be = reinterpret_cast<const uint2*>(pb)[j];
      b0 = be.x;
      e0 = be.y;
    }
    Pbeg = wave_min_u32(b0);
    Pend = wave_max_u32(e0);
  } else {
    const uint32_t* keys[2] = {T.skey_lo[k], T.skey_lo[k]};
    const uint32_t* idx[2] = {T.sidx_lo[k], T.sidx_lo[k]};
    const uint32_t x[2] = {f2key(ehi[0]), f2key(nextafterf(elo[0] - T.maxlen[k], -INFINITY))};
    const bool up[2] = {true, false};
    uint32_t res[2];
    count_2l<2>(keys, idx, x, up, T.n, T.ns, res);
    Pend = uniform_u32(res[0]);
    Pbeg = uniform_u32(res[1] + 1u);
  }
  uint32_t mycnt = 0;
  uint64_t mybase = 0, myend = 0;  // myend: segment end (write guard)
  if (FILL && qv) seg_bounds(O, gj, &mybase, &myend);
  const uint64_t mystart = mybase;
  uint64_t* __restrict__ out = O.out;
  uint32_t* __restrict__ oids = O.ids;

  const float* rec = T.rec[k];
  const float* __restrict__ bmx = T.bmax[k];
  const uint32_t* ids = T.id[k];
  uint32_t head = 0, tail = 0;
  const uint64_t lbase = MODE == kTileList && O.ids ? O.base[tile_id] : 0ull;
  const uint64_t lend = MODE == kTileList && O.ids ? O.base[tile_id + 1] : 0ull;
  // stash chunk of the wave (uniform): id, entries used, last static chunk,
  // still stashing
  uint32_t sch = tile_id * kStashStatic, sfill = 0;
  uint32_t slast = sch + kStashStatic - 1;  // last chunk the tile holds
  bool sok = STASH && sflag == 0;
  // stash: room for `tot` more entries from this wave, in the current chunk
  // and (if needed) nnew more chunks starting at `first` (static ones of the
  // tile, else counted ones from the slices); false once the stash is full
  auto stash_room = [&](uint32_t tot, uint32_t* room_out, uint32_t* first_out,
                        uint32_t* nnew_out) {
    const uint32_t room = kStashChunk - sfill;
    uint32_t first = 0, nnew = 0;
    if (room < tot) {
      nnew = (tot - room + kStashChunk - 1) / kStashChunk;
      if (sch + nnew <= slast) {
        first = sch + 1;
      } else {
        // the tile's slice first, then the following ones; the part of a
        // slice too short for the request is marked empty
        const uint32_t take = max(nnew, kStashGrab);
        if (sch < slast && lane < slast - sch) O.sused[sch + 1 + lane] = 0;
        bool got = false;
        for (uint32_t a = 0, sl = tile_id % kStashSlices; a < kStashSlices && !got;
             ++a, sl = (sl + 1) % kStashSlices) {
          const uint32_t send = O.sfirst + (sl + 1) * O.sslice;
          uint32_t f = 0;
          if (lane == 0) {
            // a slice already used up is passed over without an atomic
            f = __hip_atomic_load(O.snext + sl, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (f < send) f = atomicAdd(O.snext + sl, take);
          }
          first = uniform_u32(f);
          if (first < send && take <= send - first) {
            got = true;
          } else if (first < send && lane < send - first) {
            O.sused[first + lane] = 0;
          }
        }
        if (!got) {
          sok = false;
          if (lane == 0) atomicOr(O.snext + kStashSlices, 1u);
        } else {
          if (O.sowner && lane < take) O.sowner[first + lane] = tile_id;
          slast = first + take - 1;
        }
      }
    }
    *room_out = room;
    *first_out = first;
    *nnew_out = nnew;
    return sok;
  };
  // the stash has taken `tot` entries (room, first, nnew as stash_room gave)
  auto stash_advance = [&](uint32_t tot, uint32_t room, uint32_t first, uint32_t nnew) {
    if (nnew) {
      if (lane == 0) O.sused[sch] = kStashChunk;
      if (lane + 1 < nnew) O.sused[first + lane] = kStashChunk;
      sch = first + nnew - 1;
      sfill = tot - room - (nnew - 1) * kStashChunk;
    } else {
      sfill += tot;
    }
  };

  // tests candidates head .. head + c against the tile's updates
  auto flush = [&](uint32_t cnt) {
    wave_sync();
    const uint32_t c = uniform_u32(cnt);
    const uint32_t h0 = uniform_u32(head & (kRing - 1));  // a multiple of 64: no wrap inside
    float v[R];
    load_rec<D>(s_cand + (h0 + lane) * R, v);
    const uint32_t sid = s_cid[h0 + lane];
    if (lane >= c) {  // the last flush: nothing meets an empty slot
#pragma unroll
      for (int s = 0; s < D; ++s) {
        v[2 * s] = INFINITY;
        v[2 * s + 1] = -INFINITY;
      }
    }
    uint32_t mlo, mhi;  // this lane's update: its hits among the candidates
    test_masks<D>(ql, qh, nq, v, s_cand + h0 * R, lane, c, lane >= c, &mlo, &mhi);
    const uint32_t pcl = (uint32_t)__popc(mlo) + (uint32_t)__popc(mhi);
    uint64_t some = ballot(pcl != 0);
    if constexpr (FILL) {
      // the hits of each update go to consecutive slots of its segment; a
      // segment without room for all of them is written under a guard
      const bool tight = ballot(mybase + pcl > myend) != 0;
      while (some) {
        const uint32_t u = (uint32_t)__builtin_ctzll(some);
        some &= some - 1;
        const uint64_t m = readlane_u64((uint64_t)mhi << 32 | mlo, u);
        const uint64_t b = readlane_u64(mybase, u);
        const uint32_t r = mask_rank(m);
        bool w = lane_of(m);
        if (tight) w = w && b + r < readlane_u64(myend, u);
        if (oids) {
          if (w) (oids + b)[r] = sid;
        } else {
          const uint64_t jq = (uint64_t)readlane_u32(j, u) << 32;
          if (w) (out + b)[r] = jq | sid;
        }
      }
      mybase += pcl;
    } else {
      if constexpr (STASH) {
        // each lane stashes its own update's hits: a wave prefix of the hit
        // counts places them, one chunk request (if any) covers the flush
        // (most flushes of a sparse set have no hit at all)
        if (sok && some) {
          const uint32_t incl = wave_scan_dpp(pcl);
          const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
          uint32_t room, first, nnew;
          if (stash_room(tot, &room, &first, &nnew)) {
            uint64_t hv = (uint64_t)mhi << 32 | mlo;
            uint32_t at = incl - pcl, r = mycnt;
            while (hv) {
              const uint32_t ci = (uint32_t)__builtin_ctzll(hv);
              hv &= hv - 1;
              const uint64_t e = at < room ? (uint64_t)sch * kStashChunk + sfill + at
                                           : (uint64_t)first * kStashChunk + (at - room);
              O.skey[e] = (uint64_t)j << 32 | s_cid[h0 + ci];
              O.srank[e] = r;
              ++at;
              ++r;
            }
            stash_advance(tot, room, first, nnew);
          }
        }
      }
      mycnt += pcl;
    }
    head += c;
    wave_sync();
  };

  if (Pbeg <= Pend) {
    // blocks of 64 candidates: of the strips the range touches, kept when
    // their box meets the tile's (d > 1), or of the positions themselves,
    // kept when their maxupper reaches the tile's least lower bound
    const bool strips = D > 1 && T.sbox[k] != nullptr && Pend - Pbeg >= kStripRange;
    uint32_t c0, c1, first = Pbeg, last = Pend;
    if (strips) {
      c0 = Pbeg >> kChunkPosLog << (kChunkPosLog - kBlockLog);
      c1 = min((Pend >> kChunkPosLog << (kChunkPosLog - kBlockLog)) +
                   (1u << (kChunkPosLog - kBlockLog)),
               T.nblk) - 1u;
      first = 0u;
      last = ~0u;
      rec = T.srec[k];
      ids = T.sid[k];
    } else {
      c0 = Pbeg >> kBlockLog;
      c1 = Pend >> kBlockLog;
    }
    const float* __restrict__ box = T.sbox[k];
    // 64 blocks are looked at together; of those kept, two at a time are
    // loaded (both in flight) and staged one after the other: tested against
    // the tile's box in every dimension, the survivors appended to the ring,
    // which is flushed whenever it holds 64 and at the end
    uint32_t cb = c0, done = 0;
    uint64_t bm = 0;
    bool pick = true;
    bool second = false;
    float vA[R], vB[R];
    uint32_t idA = 0, idB = 0;
    bool inA = false, inB = false;
    while (!done) {
      if (second) {
#pragma unroll
        for (int r = 0; r < R; ++r) vA[r] = vB[r];
        idA = idB;
        inA = inB;
        second = false;
      } else {
        while (bm == 0 && cb <= c1) {
          const uint32_t c = cb + lane;
          bool keep = c <= c1;
          if (strips) {
            float b[R];
#pragma unroll
            for (int r = 0; r < R; ++r) b[r] = box[(size_t)r * T.nblk + min(c, c1)];
#pragma unroll
            for (int s = 0; s < D; ++s)
              keep = keep & (b[2 * s] <= ehi[s]) & (elo[s] <= b[2 * s + 1]);
            const uint64_t met = ballot(keep);
            if (pick && __popcll(met) > (D < 4 ? kManyBlocks : kManyBlocks4)) {
              keep = keep & meets_any<D>(b, ql, qh, nq);
              pick = 8 * __popcll(ballot(keep)) <= 7 * __popcll(met);  // (else it is dense)
            }
          } else {
            keep = keep && bmx[c] >= elo[0];
          }
          bm = ballot(keep);
          cb += kWave;
        }
        inA = false;
        if (bm != 0) {
          const uint32_t b0 = (uint32_t)__builtin_ctzll(bm);
          bm &= bm - 1;
          second = bm != 0;
          const uint32_t b1 = second ? (uint32_t)__builtin_ctzll(bm) : b0;
          if (second) bm &= bm - 1;
          const uint32_t blkA = cb - kWave + b0, blkB = cb - kWave + b1;
          const uint32_t pA = max(blkA << kBlockLog, first) + lane;
          const uint32_t pB = max(blkB << kBlockLog, first) + lane;
          inA = pA <= min((blkA << kBlockLog) + (1u << kBlockLog) - 1u, last);
          inB = second && pB <= min((blkB << kBlockLog) + (1u << kBlockLog) - 1u, last);
#pragma unroll
          for (int r = 0; r < R; ++r) vA[r] = vB[r] = 0.f;
          if (inA) {
            load_rec<D>(rec + (size_t)pA * R, vA);
            idA = ids[pA];
          }
          if (inB) {
            load_rec<D>(rec + (size_t)pB * R, vB);
            idB = ids[pB];
          }
        } else {
          done = 1;
        }
      }
      bool cnd = inA;
#pragma unroll
      for (int s = 0; s < D; ++s) cnd = cnd & (vA[2 * s] <= ehi[s]) & (elo[s] <= vA[2 * s + 1]);
      const uint64_t cm = ballot(cnd);
      if (listing) {
        if (MODE == kTileList && O.ids) {
          const uint64_t at = lbase + tail + mask_rank(cm);
          if (cnd && at < lend) O.ids[at] = idA;
        }
        tail += (uint32_t)__popcll(cm);
        continue;
      }
      if constexpr (MODE != kTileList) {
        if (cnd) {
          const uint32_t slot = (tail + mask_rank(cm)) & (kRing - 1);
          store_rec<D>(s_cand + slot * R, vA);
          s_cid[slot] = idA;
        }
        tail += (uint32_t)__popcll(cm);
        const uint32_t c = tail - head;
        if (c >= (uint32_t)kWave || (done && c != 0)) flush(min(c, (uint32_t)kWave));
      }
    }
  }
  if (STASH && sok) {
    if (lane == 0) O.sused[sch] = sfill;
    if (sch < slast && lane < slast - sch) O.sused[sch + 1 + lane] = 0;
  }
  if (listing) {
    if (O.tcand && lane == 0) {
      O.tcand[tile_id] = tail;
      uint64_t* __restrict__ slice = O.tsum + (size_t)(tile_id % kListSlices) * kListPad;
      atomicAdd((unsigned long long*)slice, (unsigned long long)tail);
      atomicMax(reinterpret_cast<uint32_t*>(slice + 1), tail);
    }
    if (MODE == kTileList) return;
  }
  if (qv) {
    if (!FILL) O.cnt[gj] = mycnt;
    else if (O.cnt) O.cnt[gj] = (uint32_t)(mybase - mystart);
  }
}

}  // namespace ddm
