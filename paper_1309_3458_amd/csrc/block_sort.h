// Stable sort of (key, value) pairs by one workgroup, all passes in LDS: for
// sets where a pass over memory is bound by its latency (8 us for 5000 keys).
#pragma once

#include "ddm_internal.h"

namespace ddm {

constexpr uint32_t kBlockSortThreads = 1024;

template <int R, typename V>
struct BlockSortLds {
  uint32_t key[kBlockSortThreads * R];
  V val[kBlockSortThreads * R];
  uint32_t wcnt[kBlockSortThreads / kWave][256];
  uint32_t wsum[4];
};

// element r of this thread
template <int R>
__device__ __forceinline__ uint32_t block_sort_index(uint32_t r) {
  return (threadIdx.x / kWave) * (R * kWave) + r * kWave + lane_id();
}

// n <= 1024 R pairs, pair i in element r of the thread with block_sort_index(r)
// == i, by the low 8 * passes bits of the key; sorted pairs are left in the same
// arrangement.  Wavefront w ranks its 64 R consecutive keys in order (a ballot
// match per round, counters of its own), so that the sort is stable.
template <int R, typename V>
__device__ __forceinline__ void block_sort(BlockSortLds<R, V>& L, uint32_t (&key)[R],
                                           uint32_t (&val)[R], uint32_t n, uint32_t passes) {
  constexpr uint32_t W = kBlockSortThreads / kWave;
  const uint32_t tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  for (uint32_t pass = 0; pass < passes; ++pass) {
    const uint32_t shift = 8u * pass;
    for (uint32_t i = lane; i < 256; i += kWave) L.wcnt[wave][i] = 0;
    uint32_t loc[R];
    // (the counters are the wavefront's own, but a lane reads what others wrote:
    // cleared above, counted in the round before)
    wave_sync();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      const bool valid = block_sort_index<R>(r) < n;
      const uint32_t dig = (key[r] >> shift) & 255u;
      const uint64_t peers = match_digit8(dig, ballot(valid));
      const uint32_t rk = mask_rank(peers);
      const uint32_t c = valid ? L.wcnt[wave][dig] : 0u;
      loc[r] = c + rk;
      wave_sync();
      if (valid && rk == 0) L.wcnt[wave][dig] = c + (uint32_t)__popcll(peers);
      wave_sync();
    }
    __syncthreads();
    // digit tid: the wavefronts' counts become offsets within the digit, then
    // the digits are placed
    uint32_t tot = 0, inc = 0;
    if (tid < 256) {
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) tot += L.wcnt[w][tid];
      inc = wave_scan_dpp(tot);
      if (lane == kWave - 1) L.wsum[wave] = inc;
    }
    __syncthreads();
    if (tid < 256) {
      uint32_t run = inc - tot;
      for (uint32_t w = 0; w < wave; ++w) run += L.wsum[w];
#pragma unroll
      for (uint32_t w = 0; w < W; ++w) {
        const uint32_t c = L.wcnt[w][tid];
        L.wcnt[w][tid] = run;
        run += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      if (block_sort_index<R>(r) < n) {
        const uint32_t at = L.wcnt[wave][(key[r] >> shift) & 255u] + loc[r];
        L.key[at] = key[r];
        L.val[at] = (V)val[r];
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      const uint32_t i = block_sort_index<R>(r);
      if (i < n) {
        key[r] = L.key[i];
        val[r] = L.val[i];
      }
    }
  }
}

}  // namespace ddm
