// Per-tree construction steps shared by the single-tree build (tree.hip) and
// the batched build (batch.hip).  Each step works on one tree (one
// dimension k of one subscription set) described by a TreeJob.
#pragma once

#include "ddm_internal.h"

namespace ddm {

struct TreeJob {
  const float* s_lo;       // the set's lower bounds, dimension-major [d][n]
  const float* s_hi;
  float* rec;              // (n+1) records of 2d floats (tree k order)
  float* maxhi;            // P+1
  float* bmax;             // C
  const uint32_t* id;      // n+1 (sorted payload at positions 1..n)
  const uint32_t* skey_lo; // n sorted keys of lo_k
  const uint32_t* skey_hi; // n sorted keys of hi_k, or null
  uint32_t* sidx_lo;       // ns samples
  uint32_t* sidx_hi;       // ns samples, or null
  uint32_t* quant;         // kQuant quantiles
  uint32_t* maxlen_bits;   // one word: bound of the lengths (float bits)
  float* srec;             // d > 1: the records strip by strip, or null
  uint32_t* sid;           // their ids
  float* sbox;             // bounding box of every block of 64 of them
  uint32_t n, d, k, P, C, H, ns;
  const float* recin;      // optional: the set as n records (lo_0, hi_0, lo_1, ...)
  uint32_t* id_out;        // optional: id and skey_lo are scratch and are also kept here
  uint32_t* key_out;
};

constexpr int kChunk = 2048;        // positions per workgroup in a maxhi pass
constexpr int kChunkLog = 11;
constexpr int kTreeThreads = 1024;  // two positions per thread

// samples of the sorted keys for two-level searches, and quantiles; index c
__device__ __forceinline__ void tree_index_item(const TreeJob& J, uint32_t c) {
  if (c < J.ns) {
    J.sidx_lo[c] = J.skey_lo[(size_t)c << 6];
    if (J.skey_hi) J.sidx_hi[c] = J.skey_hi[(size_t)c << 6];
  }
  if (c < kQuant) J.quant[c] = J.skey_lo[(uint32_t)(((uint64_t)c * J.n) / kQuant)];
}

// ---------------------------------------------------------------------------
// Strips (d > 1).  The 2048 positions of chunk c of tree k are one strip; its
// records are copied in an order that also follows the other dimensions (the
// sort-tile-recursive packing of R-trees), so that 64 consecutive ones, a
// block, lie close in every dimension, and each block gets its bounding box.
// A traversal whose updates are confined in several dimensions then skips
// blocks by their boxes instead of reading the whole range of positions
// (10^6 boxes: about 5 of 131 blocks of a tile's range stay at d = 2, alpha =
// 1, 35 of 266 at d = 3).
//   srec  strip c at records c * 2048 ..; records past its last subscription
//         are empty (lower bound +inf, upper bound -inf)
//   sbox  2d rows of nblk floats: row 2s the least lower bound, row 2s + 1
//         the greatest upper bound of record slot s
// d = 2 orders a strip by its other dimension; d = 3 sorts it by the first
// other dimension, cuts it in slabs of 512 and sorts each by the second; d =
// 4 cuts those in slabs of 128, sorted by the third.  The order is by the
// lower bound in steps of 1/2048 of the strip's extent (1/512 and 1/128 in
// the slabs); any order is correct.
//
// Each dimension is one counting sort in LDS over 2048 bins (an atomic per
// record ranks it in its bin, one scan places the bins), a few barriers in
// all; a bitonic network over the same keys took 35 us longer at 5*10^5
// squares (tree pass 61 us against 32).
// ---------------------------------------------------------------------------
constexpr uint32_t kStripLog = kChunkLog;
constexpr uint32_t kStripBlocks = kChunk / 64;
static_assert(kStripLog == 11, "traverse.h reads strips of 2048 positions");
__host__ __device__ constexpr uint32_t strip_count(uint32_t n) { return (n >> kStripLog) + 1; }

// dynamic LDS of a tree pass that writes strips: the chunk's records
// (position order), then their order
constexpr size_t strip_lds_bytes(uint32_t d) {
  return (size_t)kChunk * (sizeof(float) * 2 * d + sizeof(uint16_t));
}
extern __shared__ __align__(16) char strip_lds[];

// orders strip c (its records in LDS, in position order, empty ones where
// there is no subscription) and writes srec, sid and sbox; bins: kChunk
// words of LDS, wred: 2 words per wavefront
__device__ __forceinline__ void strip_write(const TreeJob& J, uint32_t c,
                                            uint32_t* __restrict__ bins,
                                            uint32_t* __restrict__ wred) {
  constexpr uint32_t NW = kTreeThreads / kWave;
  static_assert(kChunk == 2 * kTreeThreads, "two records per thread");
  const uint32_t D = J.d, tid = threadIdx.x, lane = lane_id(), wave = tid / kWave;
  const float* __restrict__ rec = reinterpret_cast<const float*>(strip_lds);
  uint16_t* __restrict__ order =
      reinterpret_cast<uint16_t*>(strip_lds + sizeof(float) * 2 * D * kChunk);
  for (uint32_t s = 1; s < D; ++s) {
    // records per slab: all, 512, 128
    const uint32_t slab = s == 1 ? (uint32_t)kChunk : s == 2 ? 512u : 128u;
    float mn = INFINITY, mx = -INFINITY;
    float v[2];
    uint32_t ix[2];
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q) {
      const uint32_t at = tid + q * kTreeThreads;
      ix[q] = s == 1 ? at : order[at];
      bins[at] = 0;
      // this dimension's extent over the strip (halved: no overflow)
      const float lo = rec[ix[q] * 2 * D + 2 * s];
      v[q] = 0.5f * lo;
      if (lo < INFINITY) {
        mn = fminf(mn, v[q]);
        mx = fmaxf(mx, v[q]);
      }
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    if (lane == 0) {
      wred[wave] = __float_as_uint(mn);
      wred[NW + wave] = __float_as_uint(mx);
    }
    __syncthreads();
    mn = wave_min(__uint_as_float(wred[lane % NW]));
    mx = wave_max(__uint_as_float(wred[NW + lane % NW]));
    const float sc = mx > mn ? (float)slab / (mx - mn) : 0.f;
    uint32_t bin[2], rank[2];
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q) {
      // empty records (and any NaN of invalid input) into the slab's last bin
      const float t = (v[q] - mn) * sc;
      bin[q] = ((tid + q * kTreeThreads) & ~(slab - 1u)) +
               (t < (float)slab ? (uint32_t)fmaxf(t, 0.f) : slab - 1u);
      rank[q] = atomicAdd(&bins[bin[q]], 1u);
    }
    __syncthreads();
    // exclusive scan of the bins: thread tid owns bins 2 tid and 2 tid + 1
    const uint32_t c0 = bins[2 * tid], c1 = bins[2 * tid + 1];
    const uint32_t incl = wave_scan_dpp(c0 + c1);
    if (lane == kWave - 1) wred[wave] = incl;
    __syncthreads();
    const uint32_t wt = lane < NW ? wred[lane] : 0u;
    const uint32_t before =
        (uint32_t)__builtin_amdgcn_readlane((int)(wave_scan_dpp(wt) - wt), (int)wave);
    bins[2 * tid] = before + incl - c0 - c1;
    bins[2 * tid + 1] = before + incl - c1;
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q) order[bins[bin[q]] + rank[q]] = (uint16_t)ix[q];
    __syncthreads();
  }
  const uint32_t nblk = strip_count(J.n) * kStripBlocks;
#pragma unroll
  for (uint32_t q = 0; q < 2; ++q) {
    const uint32_t slot = tid + q * kTreeThreads;
    const uint32_t ix = order[slot];
    const uint32_t p = c * kChunk + ix;
    const uint32_t blk = c * kStripBlocks + slot / 64;
    float* __restrict__ dst = J.srec + ((size_t)c * kChunk + slot) * 2 * D;
    J.sid[(size_t)c * kChunk + slot] = p >= 1 && p <= J.n ? J.id[p] : 0u;
    for (uint32_t s = 0; s < D; ++s) {
      const float2 r = *reinterpret_cast<const float2*>(rec + ix * 2 * D + 2 * s);
      *reinterpret_cast<float2*>(dst + 2 * s) = r;
      const float mn = wave_min(r.x), mx = wave_max(r.y);
      if (lane == 0) {
        J.sbox[(size_t)(2 * s) * nblk + blk] = mn;
        J.sbox[(size_t)(2 * s + 1) * nblk + blk] = mx;
      }
    }
  }
}

// Pass 0 on chunk c (2048 consecutive positions): gather the records (or,
// with GATHER false, read the records already in place, after extents have
// moved) and compute maxhi for heights 0..10 in LDS, the block maxima
// (height 5 plus the position above) and the length bound.
template <bool GATHER = true>
__device__ __forceinline__ void tree_low_chunk(const TreeJob& J, uint32_t c) {
  __shared__ float mx[kChunk];
  __shared__ uint32_t wlen[kTreeThreads / kWave];
  float* Lrec = reinterpret_cast<float*>(strip_lds);
  const uint32_t k = J.k;
  // (the grid covers the padding positions too, which have no strip)
  const bool strip = J.srec != nullptr && c < strip_count(J.n);
  const uint32_t D = J.d;
  float* __restrict__ rec = J.rec;
  const uint32_t* __restrict__ ids = J.id;
  // bound of the segment lengths in dimension k: the float difference rounded
  // to nearest, moved one float up, is >= the exact difference; lengths are
  // >= 0, so their float bits order like unsigned integers
  uint32_t lenb = 0;
  if (GATHER) {
    // every id of the thread's positions is loaded first, then every
    // record (one contiguous record per subscription with recin, else the
    // bounds of each dimension), so that there are two rounds of loads in
    // flight instead of two per position; then the records are written in
    // tree-k order (dimension k first, then the others ascending)
    constexpr uint32_t IT = kChunk / kTreeThreads;
    static_assert(kChunk % kTreeThreads == 0, "whole rounds");
    const float* __restrict__ rin = J.recin;
    uint32_t idx[IT];
    bool ok[IT];
#pragma unroll
    for (uint32_t it = 0; it < IT; ++it) {
      const uint32_t p = c * kChunk + threadIdx.x + it * kTreeThreads;
      ok[it] = p >= 1 && p <= J.n;
      idx[it] = ok[it] ? ids[p] : 0u;
    }
    float val[IT][2 * DDM_MAX_D];
#pragma unroll
    for (uint32_t it = 0; it < IT; ++it)
#pragma unroll
      for (uint32_t q = 0; q < 2 * DDM_MAX_D; ++q)
        val[it][q] = !(ok[it] && q < 2 * D) ? 0.f
                     : rin               ? rin[(size_t)idx[it] * 2 * D + q]
                     : (q & 1u)          ? J.s_hi[(size_t)(q / 2) * J.n + idx[it]]
                                         : J.s_lo[(size_t)(q / 2) * J.n + idx[it]];
#pragma unroll
    for (uint32_t it = 0; it < IT; ++it) {
      const uint32_t r = threadIdx.x + it * kTreeThreads;
      const uint32_t p = c * kChunk + r;
      float h = -INFINITY;
      if (ok[it]) {
        float* dst = rec + (size_t)p * 2 * D;
        float l0 = 0.f;
#pragma unroll
        for (uint32_t kk = 0; kk < DDM_MAX_D; ++kk) {
          if (kk >= D) continue;
          const uint32_t slot = kk == k ? 0u : (kk < k ? kk + 1u : kk);
          dst[2 * slot] = val[it][2 * kk];
          dst[2 * slot + 1] = val[it][2 * kk + 1];
          if (kk == k) {
            l0 = val[it][2 * kk];
            h = val[it][2 * kk + 1];
          }
        }
        if (J.id_out) {
          J.id_out[p] = idx[it];
          J.key_out[p - 1] = f2key(l0);
        }
        if (valid_extent(l0, h)) lenb = max(lenb, __float_as_uint(nextafterf(h - l0, INFINITY)));
      }
      if (strip) {
#pragma unroll
        for (uint32_t kk = 0; kk < DDM_MAX_D; ++kk) {
          if (kk >= D) continue;
          const uint32_t slot = kk == k ? 0u : (kk < k ? kk + 1u : kk);
          *reinterpret_cast<float2*>(Lrec + r * 2 * D + 2 * slot) =
              ok[it] ? make_float2(val[it][2 * kk], val[it][2 * kk + 1])
                     : make_float2(INFINITY, -INFINITY);
        }
      }
      mx[r] = h;
    }
  } else {
    // the records in place (extents moved): dimension k's bounds
    for (uint32_t r = threadIdx.x; r < kChunk; r += kTreeThreads) {
      const uint32_t p = c * kChunk + r;
      float h = -INFINITY;
      if (strip)
        for (uint32_t s = 0; s < D; ++s)
          *reinterpret_cast<float2*>(Lrec + r * 2 * D + 2 * s) =
              p >= 1 && p <= J.n ? *reinterpret_cast<const float2*>(rec + (size_t)p * 2 * D + 2 * s)
                                 : make_float2(INFINITY, -INFINITY);
      if (p >= 1 && p <= J.n) {
        const float* dst = rec + (size_t)p * 2 * D;
        const float l0 = dst[0];
        h = dst[1];
        if (valid_extent(l0, h)) lenb = max(lenb, __float_as_uint(nextafterf(h - l0, INFINITY)));
      }
      mx[r] = h;
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) lenb = max(lenb, (uint32_t)__shfl_xor((int)lenb, o, kWave));
  if (lane_id() == 0) wlen[threadIdx.x / kWave] = lenb;
  // Unrolled: as a loop, the compiler placed the wait for the LDS writes of one
  // height before the loop and not on its back edge, so a wavefront could pass the
  // barrier with its write still under way, and a block's maximum was now and then
  // that of a subtree not yet folded (one in some 700 replays of 256 instances).
#pragma unroll
  for (int h = 1; h < kChunkLog; ++h) {
    __syncthreads();
    if (h == 1 && threadIdx.x == 0) {
      uint32_t v = 0;
      for (int w = 0; w < kTreeThreads / kWave; ++w) v = max(v, wlen[w]);
      if (v) atomicMax(J.maxlen_bits, v);
    }
    if (h == (int)kBlockLog) {
      // heights < 6 are final and heights >= 6 still hold their own upper
      // bound: block b of the chunk is position 64b plus subtree(64b + 32)
      if (threadIdx.x < kChunk / 64) {
        const uint32_t b = threadIdx.x;
        const uint32_t blk = c * (kChunk / 64) + b;
        if (blk < J.C) J.bmax[blk] = fmaxf(mx[64 * b], mx[64 * b + 32]);
      }
      __syncthreads();
    }
    for (uint32_t r = threadIdx.x; r < kChunk; r += kTreeThreads) {
      if (r != 0 && (uint32_t)__builtin_ctz(r) == (uint32_t)h) {
        const uint32_t half = 1u << (h - 1);
        mx[r] = fmaxf(mx[r], fmaxf(mx[r - half], mx[r + half]));
      }
    }
  }
  __syncthreads();
  for (uint32_t r = threadIdx.x; r < kChunk; r += kTreeThreads) {
    const uint32_t p = c * kChunk + r;
    if (r != 0 && p <= J.P) J.maxhi[p] = mx[r];
  }
  if (strip) {
    __shared__ uint32_t wred[2 * (kTreeThreads / kWave)];
    __syncthreads();  // mx is read: its words become the bins
    strip_write(J, c, reinterpret_cast<uint32_t*>(mx), wred);
  }
}

// Pass with shift S >= 11 on chunk c: positions p = q << S (q in the chunk),
// real heights S .. S+10.  Leaves (odd q) combine the two children of height
// S-1 computed by the previous pass.
__device__ __forceinline__ void tree_high_chunk(const TreeJob& J, uint32_t c, uint32_t S) {
  __shared__ float mx[kChunk];
  const uint32_t D = J.d;
  const uint32_t qmax = J.P >> S;
  const float* __restrict__ rec = J.rec;
  float* __restrict__ maxhi = J.maxhi;
  for (uint32_t r = threadIdx.x; r < kChunk; r += kTreeThreads) {
    const uint32_t q = c * kChunk + r;
    float h = -INFINITY;
    if (r != 0 && q <= qmax) {
      const uint32_t p = q << S;
      if (p <= J.n) h = rec[(size_t)p * 2 * D + 1];
      if (q & 1u) {
        const uint32_t half = 1u << (S - 1);
        h = fmaxf(h, fmaxf(maxhi[p - half], maxhi[p + half]));
      }
    }
    mx[r] = h;
  }
#pragma unroll
  for (int h = 1; h < kChunkLog; ++h) {
    __syncthreads();
    for (uint32_t r = threadIdx.x; r < kChunk; r += kTreeThreads) {
      if (r != 0 && (uint32_t)__builtin_ctz(r) == (uint32_t)h) {
        const uint32_t half = 1u << (h - 1);
        mx[r] = fmaxf(mx[r], fmaxf(mx[r - half], mx[r + half]));
      }
    }
  }
  __syncthreads();
  for (uint32_t r = threadIdx.x; r < kChunk; r += kTreeThreads) {
    const uint32_t q = c * kChunk + r;
    if (r != 0 && q <= qmax) maxhi[q << S] = mx[r];
  }
}

}  // namespace ddm
