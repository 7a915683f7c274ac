// Dynamic DDM: both extent sets, both interval trees and the current result
// stay resident on the device, and moving extents recomputes only the pairs
// of the moved extents (the paper's dynamic scenario, Sec. IV and Sec. VI:
// one tree over the subscriptions T_S and one over the updates T_U; a moved
// update needs one query of T_S, a moved subscription one query of T_U).
//
// A move of c extents of one set:
//   1. the moved ids are marked in a bitmap (a repeated id is refused) and
//      checked with their new extents; the bitmap's prefix counts rank them,
//      so they are put in ascending order without a sort;
//   2. the resident pairs of moved ids are counted out tile by tile;
//   3. the moved extents query the other set's tree.  Its synchronization is
//      the only one: it also brings the check and the count, and nothing has
//      been changed before it;
//   4. moved updates give their columns of M directly (keys in update order);
//      moved subscriptions give their rows, which a stable sort by update id
//      turns into (update, subscription) key order;
//   5. the moved set's tree is merged (a few moves, d > 1), refitted or rebuilt
//      (ddm_tree_update), and the new extents go to the resident copy;
//   6. one pass drops the moved ids' pairs and merges the recomputed ones into
//      a new result (both lists are sorted: an element's place is its index
//      less the dropped ones before it plus the new ones before it).
// The result is always exactly the pairs of the current sets, sorted.
#include "block_sort.h"
#include "ddm_internal.h"

#include <algorithm>
#include <new>

struct ddm_dynamic {
  int device = 0;
  uint32_t n = 0, m = 0, d = 0;
  float* s_lo = nullptr;  // resident copies, dimension-major
  float* s_hi = nullptr;
  float* u_lo = nullptr;
  float* u_hi = nullptr;
  ddm_tree* ts = nullptr;  // tree over the subscriptions
  ddm_tree* tu = nullptr;  // tree over the updates
  uint64_t* pairs = nullptr;  // current result (device)
  uint64_t K = 0, cap = 0;
  hipStream_t home = nullptr;  // stream of the last call (for frees)
};

namespace ddm {

__global__ void dyn_zero_kernel(uint32_t* __restrict__ p, uint64_t count,
                                int32_t* __restrict__ flag) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0;
  if (i == 0) *flag = 0;
}

// marks the moved ids; flag |= 1 for an id out of range, |= 2 for a repeated
// id, |= 4 for an extent that is not valid
__global__ void dyn_mark_kernel(const uint32_t* __restrict__ ids, const float* __restrict__ lo,
                                const float* __restrict__ hi, uint32_t count, uint32_t d,
                                uint32_t limit, uint32_t* __restrict__ bits,
                                int32_t* __restrict__ flag) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  bool bad = false;
  for (uint32_t k = 0; k < d; ++k)
    bad = bad || !valid_extent(lo[(size_t)k * count + c], hi[(size_t)k * count + c]);
  if (bad) atomicOr(flag, 4);
  const uint32_t id = ids[c];
  if (id >= limit) {
    atomicOr(flag, 1);
    return;
  }
  const uint32_t old = atomicOr(&bits[id >> 5], 1u << (id & 31));
  if (old & (1u << (id & 31))) atomicOr(flag, 2);
}

// marked ids before each word of the bitmap, by one workgroup (16 words to a
// thread and round); and the words for the host: the flag, and the resident
// pairs that stay (*kept)
constexpr uint32_t kRankThreads = 1024, kRankWords = 16;
__global__ __launch_bounds__(kRankThreads) void dyn_rank_kernel(
    const uint32_t* __restrict__ bits, uint32_t words, uint32_t* __restrict__ before,
    const int32_t* __restrict__ flag, const uint64_t* __restrict__ kept,
    uint64_t* __restrict__ host) {
  __shared__ uint32_t wsum[2][kRankThreads / kWave];
  const uint32_t tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  if (tid == 0) {
    host[0] = (uint64_t)(uint32_t)*flag;
    host[1] = kept ? *kept : 0;
  }
  uint32_t base = 0, turn = 0;
  for (uint32_t w0 = 0; w0 < words; w0 += kRankThreads * kRankWords, turn ^= 1u) {
    const uint32_t at = w0 + tid * kRankWords;
    const bool whole = at + kRankWords <= words;  // (both arrays start at 256 bytes)
    uint32_t c[kRankWords], sum = 0;
    if (whole) {
      uint4 v[kRankWords / 4];
#pragma unroll
      for (uint32_t q = 0; q < kRankWords / 4; ++q)
        v[q] = reinterpret_cast<const uint4*>(bits + at)[q];
#pragma unroll
      for (uint32_t q = 0; q < kRankWords / 4; ++q) {
        c[4 * q] = (uint32_t)__popc(v[q].x);
        c[4 * q + 1] = (uint32_t)__popc(v[q].y);
        c[4 * q + 2] = (uint32_t)__popc(v[q].z);
        c[4 * q + 3] = (uint32_t)__popc(v[q].w);
      }
    } else {
#pragma unroll
      for (uint32_t q = 0; q < kRankWords; ++q)
        c[q] = at + q < words ? (uint32_t)__popc(bits[at + q]) : 0u;
    }
#pragma unroll
    for (uint32_t q = 0; q < kRankWords; ++q) sum += c[q];
    const uint32_t inc = wave_scan_dpp(sum);
    if (lane == kWave - 1) wsum[turn][wave] = inc;
    __syncthreads();
    const uint32_t wt = lane < kRankThreads / kWave ? wsum[turn][lane] : 0u;
    const uint32_t wi = wave_scan_dpp(wt);
    uint32_t run = base + inc - sum + (uint32_t)__builtin_amdgcn_readlane((int)(wi - wt), (int)wave);
    base += (uint32_t)__builtin_amdgcn_readlane((int)wi, kWave - 1);
#pragma unroll
    for (uint32_t q = 0; q < kRankWords; ++q) {
      const uint32_t here = c[q];
      c[q] = run;
      run += here;
    }
    if (whole) {
#pragma unroll
      for (uint32_t q = 0; q < kRankWords / 4; ++q)
        reinterpret_cast<uint4*>(before + at)[q] =
            make_uint4(c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]);
    } else {
#pragma unroll
      for (uint32_t q = 0; q < kRankWords; ++q)
        if (at + q < words) before[at + q] = c[q];
    }
  }
}

// The moved ids ascending, and their new extents in that order.  A move that the
// flag refuses leaves gaps there (a repeated id), and the host reads the flag only
// after the match: every column then becomes an extent that is not valid, so that
// the match meets nothing and stops at its own check, whatever the scratch held.
__global__ void dyn_gather_kernel(const uint32_t* __restrict__ ids, uint32_t count, uint32_t d,
                                  uint32_t limit, const float* __restrict__ new_lo,
                                  const float* __restrict__ new_hi,
                                  const uint32_t* __restrict__ bits,
                                  const uint32_t* __restrict__ before,
                                  const int32_t* __restrict__ flag, uint32_t* __restrict__ sid,
                                  float* __restrict__ glo, float* __restrict__ ghi) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  if (*flag != 0) {
    sid[c] = limit;
    for (uint32_t k = 0; k < d; ++k) {
      glo[(size_t)k * count + c] = INFINITY;
      ghi[(size_t)k * count + c] = -INFINITY;
    }
    return;
  }
  const uint32_t id = ids[c];
  const uint32_t at =
      before[id >> 5] + (uint32_t)__popc(bits[id >> 5] & ((1u << (id & 31u)) - 1u));
  sid[at] = id;
  for (uint32_t k = 0; k < d; ++k) {
    glo[(size_t)k * count + at] = new_lo[(size_t)k * count + c];
    ghi[(size_t)k * count + at] = new_hi[(size_t)k * count + c];
  }
}

// the new extents into the resident copy of the set
__global__ void dyn_scatter_kernel(const uint32_t* __restrict__ sid, uint32_t count, uint32_t d,
                                   const float* __restrict__ glo, const float* __restrict__ ghi,
                                   float* __restrict__ set_lo, float* __restrict__ set_hi,
                                   uint32_t set_count) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  const uint32_t id = sid[c];
  for (uint32_t k = 0; k < d; ++k) {
    set_lo[(size_t)k * set_count + id] = glo[(size_t)k * count + c];
    set_hi[(size_t)k * set_count + id] = ghi[(size_t)k * count + c];
  }
}

// columns of moved updates: (local << 32) | s -> (update id << 32) | s
__global__ void dyn_remap_cols_kernel(uint64_t* __restrict__ keys, uint64_t K,
                                      const uint32_t* __restrict__ sid) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K) return;
  const uint64_t k = keys[i];
  keys[i] = ((uint64_t)sid[k >> 32] << 32) | (k & 0xffffffffull);
}

// rows of moved subscriptions: (local << 32) | u -> update id, subscription
// id (split for the stable sort by update id)
__global__ void dyn_split_rows_kernel(const uint64_t* __restrict__ keys, uint64_t K,
                                      const uint32_t* __restrict__ sid,
                                      uint32_t* __restrict__ upd, uint32_t* __restrict__ sub) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= K) return;
  const uint64_t k = keys[i];
  upd[i] = (uint32_t)k;
  sub[i] = sid[k >> 32];
}

__global__ void dyn_join_kernel(const uint32_t* __restrict__ upd, const uint32_t* __restrict__ sub,
                                uint64_t K, uint64_t* __restrict__ keys) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < K) keys[i] = ((uint64_t)upd[i] << 32) | sub[i];
}

// The rows of moved subscriptions in key order at once, for up to kRowsSmall
// pairs: split, sorted by update id (stable) and joined in one workgroup, in
// place of twelve launches (10^4 pairs: 24 us in place of 53 us and their gaps).
constexpr uint32_t kRowsSmall = 16 * kBlockSortThreads;
template <int R>
__global__ __launch_bounds__(kBlockSortThreads) void dyn_rows_kernel(
    uint64_t* __restrict__ keys, uint32_t K, const uint32_t* __restrict__ sid, uint32_t passes) {
  __shared__ BlockSortLds<R, uint32_t> L;
  uint32_t key[R], val[R];
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = block_sort_index<R>(r);
    const uint64_t k = i < K ? keys[i] : 0u;
    key[r] = (uint32_t)k;
    val[r] = (uint32_t)(k >> 32);
  }
#pragma unroll
  for (uint32_t r = 0; r < R; ++r)
    if (block_sort_index<R>(r) < K) val[r] = sid[val[r]];
  block_sort<R>(L, key, val, K, passes);
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = block_sort_index<R>(r);
    if (i < K) keys[i] = ((uint64_t)key[r] << 32) | val[r];
  }
}

// The resident pairs without the moved ids' ones, tile by tile: a mask of the
// pairs that stay for every 64, how many stay before it in the tile, and how
// many of the tile.
constexpr uint32_t kPairTile = 2048, kPairThreads = 256;
constexpr uint32_t kPairRounds = kPairTile / kPairThreads, kPairWaves = kPairThreads / kWave;

__global__ __launch_bounds__(kPairThreads) void dyn_keep_kernel(
    const uint64_t* __restrict__ pairs, uint64_t K, const uint32_t* __restrict__ bits, int rows,
    uint64_t* __restrict__ mask, uint32_t* __restrict__ before, uint32_t* __restrict__ cnt) {
  __shared__ uint32_t w[kPairRounds * kPairWaves];
  const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  const uint64_t base = (uint64_t)blockIdx.x * kPairTile;
  uint32_t id[kPairRounds];
#pragma unroll
  for (uint32_t r = 0; r < kPairRounds; ++r) {
    const uint64_t i = base + r * kPairThreads + tid;
    const uint64_t k = i < K ? pairs[i] : 0u;
    id[r] = rows ? (uint32_t)k : (uint32_t)(k >> 32);
  }
#pragma unroll
  for (uint32_t r = 0; r < kPairRounds; ++r) {
    const bool stay = base + r * kPairThreads + tid < K &&
                      !((bits[id[r] >> 5] >> (id[r] & 31u)) & 1u);
    const uint64_t b = ballot(stay);
    const uint32_t q = r * kPairWaves + wave;
    if (lane == 0) {
      mask[base / 64 + q] = b;
      w[q] = (uint32_t)__popcll(b);
    }
  }
  __syncthreads();
  if (wave == 0) {
    constexpr uint32_t Q = kPairRounds * kPairWaves;
    const uint32_t v = lane < Q ? w[lane] : 0u;
    const uint32_t inc = wave_scan_dpp(v);
    if (lane < Q) before[base / 64 + lane] = inc - v;
    if (lane == Q - 1) cnt[blockIdx.x] = inc;
  }
}

// elements of sorted v[lo, hi) below x, plus lo
__device__ __forceinline__ uint64_t count_below(const uint64_t* __restrict__ v, uint64_t lo,
                                                uint64_t hi, uint64_t x) {
  while (lo < hi) {
    const uint64_t mid = (lo + hi) >> 1;
    if (v[mid] < x) lo = mid + 1;
    else hi = mid;
  }
  return lo;
}

// the same from 0, by one wavefront (64 probes at a time)
__device__ __forceinline__ uint64_t wave_count_below(const uint64_t* __restrict__ v, uint64_t len,
                                                     uint64_t x) {
  uint64_t at = 0;
  while (len) {
    const uint64_t step = (len + kWave - 1) / kWave;
    const uint64_t o = lane_id() * step + step - 1;
    const bool less = o < len && v[at + o] < x;
    const uint64_t full = (uint64_t)__popcll(ballot(less)) * step;
    at += full;
    len = min(step - 1, len - full);
  }
  return at;
}

// The new result: workgroups 0 .. tiles-1 take a tile of the old pairs each (the
// new ones that fall into it are found by two searches and held in LDS), the
// others 256 new pairs each.  The compaction and the merge were three passes
// over the result before (39 us for 10^6 pairs, 16 with this).
constexpr uint32_t kPairCache = 1024;
__global__ __launch_bounds__(kPairThreads) void dyn_merge_kernel(
    const uint64_t* __restrict__ pairs, uint64_t K, const uint64_t* __restrict__ mask,
    const uint32_t* __restrict__ before, const uint64_t* __restrict__ tile_off, uint32_t tiles,
    const uint64_t* __restrict__ fresh, uint64_t F, uint64_t* __restrict__ out) {
  const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  if (blockIdx.x >= tiles) {
    const uint64_t q = (uint64_t)(blockIdx.x - tiles) * kPairThreads + tid;
    if (q >= F) return;
    const uint64_t x = fresh[q];
    const uint64_t j = count_below(pairs, 0, K, x);
    uint64_t kept;
    if (j == K)
      kept = tile_off ? tile_off[tiles] : 0;
    else
      kept = tile_off[j / kPairTile] + before[j / 64] +
             (uint64_t)__popcll(mask[j / 64] & ((1ull << (j & 63u)) - 1ull));
    out[q + kept] = x;
    return;
  }
  __shared__ uint64_t cache[kPairCache];
  __shared__ uint64_t bound[2];
  const uint64_t base = (uint64_t)blockIdx.x * kPairTile;
  const uint64_t off = tile_off[blockIdx.x];
  uint64_t key[kPairRounds];
#pragma unroll
  for (uint32_t r = 0; r < kPairRounds; ++r) {
    const uint64_t i = base + r * kPairThreads + tid;
    key[r] = i < K ? pairs[i] : ~0ull;
  }
  if (wave < 2) {
    const uint64_t at = base + wave * (uint64_t)kPairTile;
    const uint64_t v = at < K ? wave_count_below(fresh, F, pairs[at]) : F;
    if (lane == 0) bound[wave] = v;
  }
  __syncthreads();
  const uint64_t i0 = bound[0], i1 = bound[1];
  const bool cached = i1 - i0 <= kPairCache;
  if (cached)
    for (uint64_t q = i0 + tid; q < i1; q += kPairThreads) cache[q - i0] = fresh[q];
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < kPairRounds; ++r) {
    const uint64_t w = base / 64 + r * kPairWaves + wave;
    const uint64_t m = mask[w];
    if (!((m >> lane) & 1u)) continue;
    const uint64_t at = cached ? i0 + count_below(cache, 0, i1 - i0, key[r])
                               : count_below(fresh, i0, i1, key[r]);
    out[off + before[w] + mask_rank(m) + at] = key[r];
  }
}

static unsigned blocks(uint64_t count) { return (unsigned)((count + 255) / 256); }

// stable LSD radix sort of `count` (key, value) u32 pairs by the key's
// passes (8 bits each); the result lands in buffer index passes & 1
static ddm_status sort_pairs(uint32_t* const (&k)[2], uint32_t* const (&v)[2], uint32_t count,
                             uint32_t passes, hipStream_t s) {
  if (passes == 0 || count == 0) return DDM_OK;
  const uint32_t ntiles = (count + kSortTile - 1) / kSortTile;
  Scratch sc(s);
  sc.reserve(sizeof(SortArr));
  sc.reserve(sizeof(uint32_t) * ntiles);
  sc.reserve(sizeof(uint32_t) * 256 * (size_t)ntiles);
  if (!sc.commit()) return DDM_E_NOMEM;
  SortArr* arr = sc.take<SortArr>(1);
  uint32_t* tile_map = sc.take<uint32_t>(ntiles);
  uint32_t* hist = sc.take<uint32_t>(256 * (size_t)ntiles);
  if (!sc.fits()) return scratch_overrun("dynamic sort");
  SortArr h{{k[0], k[1]}, {v[0], v[1]}, count, 0};
  ddm_status r = sort_setup_small(&h, 1, arr, tile_map, ntiles, s);
  if (r != DDM_OK) return r;
  return radix_sort_batch(arr, 1, tile_map, ntiles, hist, 0, (int)passes, s);
}

static uint32_t passes_for(uint32_t max_value) {
  uint32_t p = 0;
  for (uint32_t v = max_value; v; v >>= 8) ++p;
  return p;
}

// the K pairs of the moved extents (ids sid) out of a match against the other
// set's tree, as (update << 32) | subscription keys sorted ascending, in keys;
// rows: the moved extents are subscriptions, and keys has room for 16 more
// bytes per pair if K > kRowsSmall
static ddm_status recomputed_keys(const ddm_dynamic* dy, bool rows, const uint32_t* sid,
                                  uint64_t* keys, uint64_t K, hipStream_t s) {
  if (!rows) {
    dyn_remap_cols_kernel<<<blocks(K), 256, 0, s>>>(keys, K, sid);
    DDM_LAUNCHED("dyn_remap_cols_kernel");
    return DDM_OK;
  }
  // (subscription, update) order -> (update, subscription) order: a stable
  // sort by update id keeps each update's subscriptions ascending
  const uint32_t passes = passes_for(dy->m - 1);
  if (K <= kRowsSmall) {
#define DDM_ROWS(R) \
  dyn_rows_kernel<R><<<1, kBlockSortThreads, 0, s>>>(keys, (uint32_t)K, sid, passes)
    // (a key's round costs the same whether it is there or not; sizes in between take
    // the next one, at most a quarter more rounds from 8 on)
    const uint32_t need = (uint32_t)((K + kBlockSortThreads - 1) / kBlockSortThreads);
    if (need <= 1)
      DDM_ROWS(1);
    else if (need <= 2)
      DDM_ROWS(2);
    else if (need <= 4)
      DDM_ROWS(4);
    else if (need <= 8)
      DDM_ROWS(8);
    else if (need <= 10)
      DDM_ROWS(10);
    else if (need <= 12)
      DDM_ROWS(12);
    else
      DDM_ROWS(16);
#undef DDM_ROWS
    DDM_LAUNCHED("dyn_rows_kernel");
    return DDM_OK;
  }
  uint32_t* base = (uint32_t*)(keys + K);
  uint32_t* const ku[2] = {base, base + K};
  uint32_t* const vs[2] = {base + 2 * K, base + 3 * K};
  dyn_split_rows_kernel<<<blocks(K), 256, 0, s>>>(keys, K, sid, ku[0], vs[0]);
  DDM_LAUNCHED("dyn_split_rows_kernel");
  const ddm_status r = sort_pairs(ku, vs, (uint32_t)K, passes, s);
  if (r != DDM_OK) return r;
  dyn_join_kernel<<<blocks(K), 256, 0, s>>>(ku[passes & 1], vs[passes & 1], K, keys);
  DDM_LAUNCHED("dyn_join_kernel");
  return DDM_OK;
}

}  // namespace ddm

using namespace ddm;

extern "C" ddm_status ddm_dynamic_create(const float* sub_lo, const float* sub_hi, uint32_t n,
                                         const float* upd_lo, const float* upd_hi, uint32_t m,
                                         uint32_t d, void* stream, ddm_dynamic** out) {
  set_detail("");
  if (!out || d < 1 || d > DDM_MAX_D || (n && (!sub_lo || !sub_hi)) ||
      (m && (!upd_lo || !upd_hi)) || n >= 0x80000000u || m >= 0x80000000u) {
    set_detail("ddm_dynamic_create: bad argument");
    return DDM_E_INVALID_ARG;
  }
  *out = nullptr;
  hipStream_t s = (hipStream_t)stream;
  ddm_dynamic* dy = new (std::nothrow) ddm_dynamic();
  if (!dy) return DDM_E_NOMEM;
  DDM_HIP(hipGetDevice(&dy->device));
  dy->n = n;
  dy->m = m;
  dy->d = d;
  dy->home = s;
  const size_t sb = sizeof(float) * d * (size_t)std::max(n, 1u);
  const size_t ub = sizeof(float) * d * (size_t)std::max(m, 1u);
  dy->s_lo = (float*)dev_alloc(sb, s);
  dy->s_hi = (float*)dev_alloc(sb, s);
  dy->u_lo = (float*)dev_alloc(ub, s);
  dy->u_hi = (float*)dev_alloc(ub, s);
  auto fail = [&](ddm_status r) {
    ddm_dynamic_free(dy);
    return r;
  };
  if (!dy->s_lo || !dy->s_hi || !dy->u_lo || !dy->u_hi) {
    set_detail("ddm_dynamic_create: device allocation failed");
    return fail(DDM_E_NOMEM);
  }
  if (n) {
    DDM_HIP(hipMemcpyAsync(dy->s_lo, sub_lo, sizeof(float) * d * (size_t)n,
                           hipMemcpyDeviceToDevice, s));
    DDM_HIP(hipMemcpyAsync(dy->s_hi, sub_hi, sizeof(float) * d * (size_t)n,
                           hipMemcpyDeviceToDevice, s));
  }
  if (m) {
    DDM_HIP(hipMemcpyAsync(dy->u_lo, upd_lo, sizeof(float) * d * (size_t)m,
                           hipMemcpyDeviceToDevice, s));
    DDM_HIP(hipMemcpyAsync(dy->u_hi, upd_hi, sizeof(float) * d * (size_t)m,
                           hipMemcpyDeviceToDevice, s));
  }
  ddm_status r = ddm_build(dy->s_lo, dy->s_hi, n, d, stream, &dy->ts);
  if (r != DDM_OK) return fail(r);
  r = ddm_build(dy->u_lo, dy->u_hi, m, d, stream, &dy->tu);
  if (r != DDM_OK) return fail(r);
  r = ddm_tree_check(dy->tu);
  if (r != DDM_OK) return fail(r);
  uint64_t K = 0;
  ddm_pending* pend = nullptr;
  r = ddm_match_begin(dy->ts, dy->u_lo, dy->u_hi, m, &K, stream, nullptr, &pend);
  if (r != DDM_OK) return fail(r);
  dy->cap = std::max<uint64_t>(K, 1);
  dy->pairs = (uint64_t*)dev_alloc(sizeof(uint64_t) * dy->cap, s);
  if (!dy->pairs) {
    ddm_match_abort(pend);
    set_detail("ddm_dynamic_create: device allocation failed");
    return fail(DDM_E_NOMEM);
  }
  r = ddm_match_finish(pend, dy->pairs, dy->cap);
  if (r != DDM_OK) return fail(r);
  dy->K = K;
  *out = dy;
  return DDM_OK;
}

extern "C" ddm_status ddm_dynamic_move(ddm_dynamic* dy, uint32_t set, const uint32_t* ids,
                                       const float* new_lo, const float* new_hi, uint32_t count,
                                       void* stream, uint64_t* out_count) {
  set_detail("");
  if (!dy || set > DDM_DYNAMIC_UPDATES || (count && (!ids || !new_lo || !new_hi))) {
    set_detail("ddm_dynamic_move: bad argument");
    return DDM_E_INVALID_ARG;
  }
  if (out_count) *out_count = dy->K;
  if (count == 0) return DDM_OK;
  int cur = -1;
  DDM_HIP(hipGetDevice(&cur));
  if (cur != dy->device) {
    set_detail("ddm_dynamic_move: the current device is not the object's device");
    return DDM_E_INVALID_ARG;
  }
  const bool rows = set == DDM_DYNAMIC_SUBSCRIPTIONS;
  const uint32_t limit = rows ? dy->n : dy->m;
  if (count > limit) {
    set_detail("ddm_dynamic_move: more moves than extents in the set");
    return DDM_E_INVALID_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  dy->home = s;
  const uint32_t d = dy->d;
  const uint64_t K = dy->K;
  if (K >= (1ull << 32)) {
    set_detail("ddm_dynamic_move: more than 2^32 - 1 resident pairs");
    return DDM_E_INVALID_ARG;
  }
  ddm_tree* const own = rows ? dy->ts : dy->tu;
  const ddm_tree* const other = rows ? dy->tu : dy->ts;
  const bool merge = tree_move_ok(own, count);
  const uint32_t words = (limit + 31) / 32;
  const uint32_t tiles = (uint32_t)((K + kPairTile - 1) / kPairTile);
  const size_t blk64 = (size_t)tiles * (kPairTile / 64);
  Scratch sc(s);
  sc.reserve(sizeof(uint32_t) * words);               // bitmap
  sc.reserve(sizeof(uint32_t) * words);               // marked before each word
  sc.reserve(sizeof(int32_t));                        // flag
  sc.reserve(sizeof(uint32_t) * count);               // moved ids, ascending
  sc.reserve(sizeof(float) * d * (size_t)count);      // their extents
  sc.reserve(sizeof(float) * d * (size_t)count);
  sc.reserve(merge ? sizeof(uint32_t) * tree_move_words(own, count) : 1);
  sc.reserve(sizeof(uint64_t) * (blk64 + 1));         // resident pairs: masks,
  sc.reserve(sizeof(uint32_t) * (blk64 + 1));         // counts before them,
  sc.reserve(sizeof(uint32_t) * (tiles + 1));         // counts of the tiles
  sc.reserve(sizeof(uint64_t) * ((size_t)tiles + 1)); // and their sums
  sc.reserve(sizeof(uint64_t) * scan_tmp_words(tiles));
  if (!sc.commit()) return DDM_E_NOMEM;
  uint32_t* bits = sc.take<uint32_t>(words);
  uint32_t* before = sc.take<uint32_t>(words);
  int32_t* flag = sc.take<int32_t>(1);
  uint32_t* sid = sc.take<uint32_t>(count);
  float* glo = sc.take<float>((size_t)d * count);
  float* ghi = sc.take<float>((size_t)d * count);
  TreeMove M{sid, glo, ghi, bits, count, nullptr};
  if (merge)
    M.words = sc.take<uint32_t>(tree_move_words(own, count));
  else
    (void)sc.take<char>(1);
  uint64_t* mask = sc.take<uint64_t>(blk64 + 1);
  uint32_t* mask_before = sc.take<uint32_t>(blk64 + 1);
  uint32_t* tile_cnt = sc.take<uint32_t>((size_t)tiles + 1);
  uint64_t* tile_off = sc.take<uint64_t>((size_t)tiles + 1);
  uint64_t* stmp = sc.take<uint64_t>(scan_tmp_words(tiles));
  if (!sc.fits()) return scratch_overrun("ddm_dynamic_move");
  uint64_t* hw = nullptr;
  ddm_status r = host_words(&hw);
  if (r != DDM_OK) return r;
  hw += kHostWordsMove;
  // 1., 2. nothing of the object is written until the host has read the flag
  dyn_zero_kernel<<<blocks(words), 256, 0, s>>>(bits, words, flag);
  DDM_LAUNCHED("dyn_zero_kernel");
  dyn_mark_kernel<<<blocks(count), 256, 0, s>>>(ids, new_lo, new_hi, count, d, limit, bits, flag);
  DDM_LAUNCHED("dyn_mark_kernel");
  if (tiles) {
    dyn_keep_kernel<<<tiles, kPairThreads, 0, s>>>(dy->pairs, K, bits, rows ? 1 : 0, mask,
                                                   mask_before, tile_cnt);
    DDM_LAUNCHED("dyn_keep_kernel");
    r = scan_u32_u64(tile_cnt, tile_off, tiles, stmp, s);
    if (r != DDM_OK) return r;
  }
  dyn_rank_kernel<<<1, kRankThreads, 0, s>>>(bits, words, before, flag,
                                             tiles ? tile_off + tiles : nullptr, hw);
  DDM_LAUNCHED("dyn_rank_kernel");
  dyn_gather_kernel<<<blocks(count), 256, 0, s>>>(ids, count, d, limit, new_lo, new_hi, bits,
                                                  before, flag, sid, glo, ghi);
  DDM_LAUNCHED("dyn_gather_kernel");
  if (merge) {
    r = tree_move_sort(own, M, s);
    if (r != DDM_OK) return r;
  }
  // 3. the moved extents' pairs against the other set's tree
  uint64_t F = 0;
  ddm_pending* pend = nullptr;
  r = ddm_match_begin(other, glo, ghi, count, &F, stream, nullptr, &pend);
  const hipError_t sync = hipStreamSynchronize(s);  // (a match without a tree has not waited)
  if (sync != hipSuccess) {
    ddm_match_abort(pend);
    return hip_fail(sync, "hipStreamSynchronize", __FILE__, __LINE__);
  }
  if (hw[0]) {
    ddm_match_abort(pend);
    set_detail(hw[0] & 1   ? "ddm_dynamic_move: id out of range"
               : hw[0] & 2 ? "ddm_dynamic_move: an id appears more than once"
                           : "ddm_dynamic_move: NaN/inf or lo > hi in the new extents");
    return DDM_E_INVALID_INPUT;
  }
  if (r != DDM_OK) return r;
  if (F >= (1ull << 32)) {
    ddm_match_abort(pend);
    set_detail("dynamic move: more than 2^32 - 1 recomputed pairs");
    return DDM_E_INVALID_ARG;
  }
  const uint64_t A = hw[1], total = A + F;
  // 4. the recomputed pairs, and the memory of the new result
  uint64_t* fresh = nullptr;
  char* fresh_mem = nullptr;
  if (F) {
    fresh_mem = dev_alloc(sizeof(uint64_t) * F + (rows && F > kRowsSmall ? 16 * F + 1024 : 0), s);
    fresh = (uint64_t*)fresh_mem;
  }
  const uint64_t cap = std::max(dy->cap, total);
  uint64_t* result = (uint64_t*)dev_alloc(sizeof(uint64_t) * cap, s);
  auto fail = [&](ddm_status st) {
    if (fresh_mem) dev_free(fresh_mem, s);
    if (result) dev_free((char*)result, s);
    return st;
  };
  if ((F && !fresh) || !result) {
    ddm_match_abort(pend);
    set_detail("dynamic move: device allocation failed");
    return fail(DDM_E_NOMEM);
  }
  r = ddm_match_finish(pend, fresh, F);
  if (r == DDM_OK && F) r = recomputed_keys(dy, rows, sid, fresh, F, s);
  if (r != DDM_OK) return fail(r);
  // 5. the tree and the resident copy
  r = merge ? tree_move_apply(own, M, s)
            : ddm_tree_update(own, ids, new_lo, new_hi, count, stream, nullptr);
  if (r != DDM_OK) return fail(r);
  dyn_scatter_kernel<<<blocks(count), 256, 0, s>>>(sid, count, d, glo, ghi,
                                                   rows ? dy->s_lo : dy->u_lo,
                                                   rows ? dy->s_hi : dy->u_hi, limit);
  DDM_LAUNCHED("dyn_scatter_kernel");
  // 6. the new result
  const uint64_t groups = tiles + (F + kPairThreads - 1) / kPairThreads;
  if (groups) {
    dyn_merge_kernel<<<(unsigned)groups, kPairThreads, 0, s>>>(
        dy->pairs, K, mask, mask_before, tiles ? tile_off : nullptr, tiles, fresh, F, result);
    DDM_LAUNCHED("dyn_merge_kernel");
  }
  dev_free((char*)dy->pairs, s);
  dy->pairs = result;
  dy->cap = cap;
  dy->K = total;
  if (fresh_mem) dev_free(fresh_mem, s);
  if (out_count) *out_count = total;
  return DDM_OK;
}

extern "C" ddm_status ddm_dynamic_result(const ddm_dynamic* dy, const uint64_t** pairs,
                                         uint64_t* count) {
  if (!dy || !pairs || !count) return DDM_E_INVALID_ARG;
  *pairs = dy->pairs;
  *count = dy->K;
  return DDM_OK;
}

extern "C" void ddm_dynamic_free(ddm_dynamic* dy) {
  if (!dy) return;
  if (dy->ts) ddm_tree_free(dy->ts);
  if (dy->tu) ddm_tree_free(dy->tu);
  hipStream_t s = dy->home;
  if (dy->pairs) dev_free((char*)dy->pairs, s);
  if (dy->s_lo) dev_free((char*)dy->s_lo, s);
  if (dy->s_hi) dev_free((char*)dy->s_hi, s);
  if (dy->u_lo) dev_free((char*)dy->u_lo, s);
  if (dy->u_hi) dev_free((char*)dy->u_hi, s);
  delete dy;
}
