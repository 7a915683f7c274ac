// Interval tree construction on the device (Sec. IV, Interval-Tree-Create).
//
// The paper builds an augmented AVL tree by insertion.  Here the tree over a
// static subscription set is flat and implicit: segments sorted by lower
// bound occupy in-order positions 1..n of a complete binary tree with
// P = 2^H - 1 >= n positions, where position p has height ctz(p), children
// p -/+ 2^(h-1) and subtree span [p - 2^h + 1, p + 2^h - 1].  The order is
// the paper's (lower bound first); equal lower bounds keep subscription id
// order (stable sort) instead of the upper-bound tie-break, which changes
// no query result.  Each position stores maxupper of its subtree, computed
// bottom-up; minlower is the lower bound at the leftmost position of the
// subtree and needs no storage.  Positions beyond n are padding, recognised
// by index only.
#include "block_sort.h"
#include "ddm_internal.h"
#include "tree_dev.h"

#include <algorithm>
#include <mutex>
#include <new>

struct ddm_tree {
  int device = 0;
  hipStream_t stream = nullptr;
  uint32_t n = 0, d = 0, H = 0, P = 0;
  char* block = nullptr;  // one device allocation for everything below
  float* rec[DDM_MAX_D] = {};
  float* maxhi[DDM_MAX_D] = {};
  uint32_t* id[DDM_MAX_D] = {};
  uint32_t* skey_lo[DDM_MAX_D] = {};
  uint32_t* skey_hi[DDM_MAX_D] = {};
  float* bmax[DDM_MAX_D] = {};
  uint32_t* sidx_lo[DDM_MAX_D] = {};
  uint32_t* sidx_hi[DDM_MAX_D] = {};
  uint32_t* quant[DDM_MAX_D] = {};
  float* srec[DDM_MAX_D] = {};  // d > 1: strips (tree_dev.h)
  uint32_t* sid[DDM_MAX_D] = {};
  float* sbox[DDM_MAX_D] = {};
  float* rid = nullptr;  // the set as records by id
  uint32_t ns = 0;              // ceil(n / 64) search samples
  uint32_t C = 0;               // blocks of 64 positions
  float* maxlen = nullptr;      // d floats (device)
  float* fstat = nullptr;       // feature statistics (learned sizing)
  uint32_t* fcum = nullptr;
  uint32_t* sat = nullptr;
  int32_t* flag = nullptr;  // device: nonzero if a coordinate was invalid
  // feature statistics are computed on the first learned match (they are
  // not needed otherwise); `fstats_ready` marks them enqueued on the stream
  // of that match, `fstats_event` lets other streams wait for them
  std::mutex fmu;
  bool fstats_ready = false;
  hipEvent_t fstats_event = nullptr;
};

namespace ddm {

TreeDev tree_dev(const ddm_tree* t) {
  TreeDev T{};
  for (uint32_t k = 0; k < t->d; ++k) {
    T.rec[k] = t->rec[k];
    T.maxhi[k] = t->maxhi[k];
    T.id[k] = t->id[k];
    T.skey_lo[k] = t->skey_lo[k];
    T.skey_hi[k] = t->skey_hi[k];
    T.bmax[k] = t->bmax[k];
    T.sidx_lo[k] = t->sidx_lo[k];
    T.sidx_hi[k] = t->sidx_hi[k];
    T.quant[k] = t->quant[k];
    T.srec[k] = t->srec[k];
    T.sid[k] = t->sid[k];
    T.sbox[k] = t->sbox[k];
  }
  T.nblk = t->d > 1 ? strip_count(t->n) * kStripBlocks : 0u;
  T.rid = t->rid;
  T.ns = t->ns;
  T.maxlen = t->maxlen;
  T.n = t->n;
  T.d = t->d;
  T.H = t->H;
  return T;
}

FeatDev tree_feat(const ddm_tree* t) { return FeatDev{t->fstat, t->fcum, t->sat, t->n, t->d}; }
const int32_t* tree_flag(const ddm_tree* t) { return t->flag; }
uint32_t tree_n(const ddm_tree* t) { return t->n; }
uint32_t tree_d(const ddm_tree* t) { return t->d; }
int tree_device(const ddm_tree* t) { return t->device; }

// clears what a build adds to: the flag, the length bounds and the sort's tables
__global__ __launch_bounds__(256) void build_zero_kernel(int32_t* __restrict__ flag,
                                                         uint32_t* __restrict__ maxlen_bits,
                                                         uint32_t d, OsScratch S) {
  const size_t g = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = g; i < S.nhist; i += stride) S.ghist[i] = 0;
  for (size_t i = g; i < S.nstatus; i += stride) S.status[i] = 0;
  if (g < 4) S.ctr[g] = 0;
  if (g < d) maxlen_bits[g] = 0;
  if (g == 0) *flag = 0;
}

// Validity, order-preserving keys, identity payload (id arrays shifted by one
// so that the sorted payload lands directly at positions 1..n), and the set
// as n records (lo_0, hi_0, lo_1, hi_1, ...), which the tree pass gathers one
// by one.  The digits of the keys are counted here too, while the keys are in
// registers: a pass over the keys for the sort's histograms and its launch
// cost 9 us more at 5*10^5 squares.
constexpr uint32_t kKeyThreads = 256, kKeyItems = 8;

template <int D>
__global__ __launch_bounds__(kKeyThreads) void build_keys_kernel(
    const float* __restrict__ lo, const float* __restrict__ hi, uint32_t n,
    uint32_t* __restrict__ klo, uint32_t* __restrict__ khi, uint32_t* __restrict__ id_base,
    int32_t* __restrict__ flag, float* __restrict__ recin, uint32_t* __restrict__ ghist) {
  constexpr int A = D == 1 ? 2 : D;  // arrays sorted: lower bounds, for d = 1 the upper ones too
  __shared__ uint32_t h[A * 4][256];
  const uint32_t tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < A * 4; ++q) h[q][tid] = 0;
  const uint32_t base = blockIdx.x * (kKeyThreads * kKeyItems) + tid;
  float a[kKeyItems][D], b[kKeyItems][D];
#pragma unroll
  for (uint32_t r = 0; r < kKeyItems; ++r) {
    const uint32_t i = base + r * kKeyThreads;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      a[r][k] = i < n ? lo[(size_t)k * n + i] : 0.f;
      b[r][k] = i < n ? hi[(size_t)k * n + i] : 0.f;
    }
  }
  __syncthreads();
  bool bad = false;
#pragma unroll
  for (uint32_t r = 0; r < kKeyItems; ++r) {
    const uint32_t i = base + r * kKeyThreads;
    if (i < n) {
#pragma unroll
      for (int k = 0; k < D; ++k) {
        bad = bad || !valid_extent(a[r][k], b[r][k]);
        const uint32_t kl = f2key(a[r][k]);
        klo[(size_t)k * n + i] = kl;
        id_base[(size_t)k * (n + 1) + 1 + i] = i;
        *reinterpret_cast<float2*>(recin + ((size_t)i * D + k) * 2) = make_float2(a[r][k], b[r][k]);
#pragma unroll
        for (int p = 0; p < 4; ++p) atomicAdd(&h[k * 4 + p][(kl >> (8 * p)) & 255u], 1u);
        if (D == 1) {
          const uint32_t kh = f2key(b[r][k]);
          khi[i] = kh;
#pragma unroll
          for (int p = 0; p < 4; ++p) atomicAdd(&h[(A - 1) * 4 + p][(kh >> (8 * p)) & 255u], 1u);
        }
      }
    }
  }
  if (ballot(bad) != 0 && lane_id() == 0) atomicOr(flag, 1);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < A * 4; ++q) {
    const uint32_t c = h[q][tid];
    if (c) atomicAdd(&ghist[q * 256 + tid], c);
  }
}

// Small sets: keys and sort in one kernel, one workgroup per sorted array, in
// place of the eight launches of the general path (5000 segments: 41 us of
// kernels and their gaps against 17).
constexpr uint32_t kSmallThreads = kBlockSortThreads, kSmallMax = 8192;

template <int R>
__global__ __launch_bounds__(kSmallThreads) void build_small_kernel(
    const float* __restrict__ lo, const float* __restrict__ hi, uint32_t n, uint32_t d,
    uint32_t* __restrict__ klo, uint32_t* __restrict__ khi, uint32_t* __restrict__ id_base,
    int32_t* __restrict__ flag, uint32_t* __restrict__ maxlen_bits, float* __restrict__ recin) {
  __shared__ BlockSortLds<R, uint16_t> L;
  __shared__ uint32_t sbad;
  const uint32_t tid = threadIdx.x;
  // dimension blockIdx.x, or (d = 1, second workgroup) the upper bounds
  const uint32_t k = blockIdx.x < d ? blockIdx.x : 0u;
  const bool upper = blockIdx.x >= d;
  if (tid == 0) sbad = 0;
  uint32_t key[R], val[R];
  bool bad = false;
  {
    float a[R], b[R];
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      const uint32_t i = block_sort_index<R>(r);
      a[r] = i < n ? lo[(size_t)k * n + i] : 0.f;
      b[r] = i < n ? hi[(size_t)k * n + i] : 0.f;
    }
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) {
      const uint32_t i = block_sort_index<R>(r);
      key[r] = f2key(upper ? b[r] : a[r]);
      val[r] = i;
      bad = bad || !valid_extent(a[r], b[r]);
      if (!upper && i < n)
        *reinterpret_cast<float2*>(recin + ((size_t)i * d + k) * 2) = make_float2(a[r], b[r]);
    }
  }
  // the first workgroup looks at every dimension, so that the flag has one writer
  if (blockIdx.x == 0)
    for (uint32_t kk = 1; kk < d; ++kk) {
      float a[R], b[R];
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) {
        const uint32_t i = block_sort_index<R>(r);
        a[r] = i < n ? lo[(size_t)kk * n + i] : 0.f;
        b[r] = i < n ? hi[(size_t)kk * n + i] : 0.f;
      }
#pragma unroll
      for (uint32_t r = 0; r < R; ++r) bad = bad || !valid_extent(a[r], b[r]);
    }
  __syncthreads();
  if (bad) sbad = 1;
  block_sort<R>(L, key, val, n, 4);
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = block_sort_index<R>(r);
    if (i < n) {
      if (upper) {
        khi[i] = key[r];
      } else {
        klo[(size_t)k * n + i] = key[r];
        id_base[(size_t)k * (n + 1) + 1 + i] = val[r];
      }
    }
  }
  if (tid == 0) {
    if (!upper) maxlen_bits[k] = 0;
    if (blockIdx.x == 0) *flag = sbad ? 1 : 0;
  }
}

// up to DDM_MAX_D tree jobs passed by value (one build)
struct TreeJobs {
  TreeJob j[DDM_MAX_D];
};

__global__ void flag_zero_kernel(int32_t* __restrict__ flag) {
  if (threadIdx.x == 0) *flag = 0;
}

// job blockIdx.y, chunk blockIdx.x - ig; the first ig workgroups take the samples
// and quantiles instead, one item to a thread (they need the sorted keys only, so
// their loads run beside the other workgroups': 5 us less than a kernel of their
// own at 5*10^5; all items in one workgroup took 24 us where the pass takes 12)
__device__ __forceinline__ bool tree_index_group(const TreeJob& J, uint32_t ig) {
  if (blockIdx.x >= ig) return false;
  tree_index_item(J, blockIdx.x * kTreeThreads + threadIdx.x);
  return true;
}

__global__ __launch_bounds__(kTreeThreads) void tree_low_kernel(TreeJobs J, uint32_t ig) {
  if (tree_index_group(J.j[blockIdx.y], ig)) return;
  tree_low_chunk(J.j[blockIdx.y], blockIdx.x - ig);
}

// the same pass over records already in place (extents moved)
__global__ __launch_bounds__(kTreeThreads) void tree_refit_kernel(TreeJobs J, uint32_t ig) {
  if (tree_index_group(J.j[blockIdx.y], ig)) return;
  tree_low_chunk<false>(J.j[blockIdx.y], blockIdx.x - ig);
}

__global__ __launch_bounds__(kTreeThreads) void tree_high_kernel(TreeJobs J, uint32_t S) {
  tree_high_chunk(J.j[blockIdx.y], blockIdx.x, S);
}

static size_t al(size_t b) { return (b + 255) & ~size_t(255); }

// device bytes of a tree over n subscriptions in d dimensions (one block)
size_t tree_bytes_estimate(uint32_t n, uint32_t d) {
  if (n == 0) return 0;
  uint32_t H = 0;
  while (H < 32 && ((1ull << H) - 1) < n) ++H;
  const uint64_t P = (1ull << H) - 1;
  const size_t rec_b = al(sizeof(float) * (size_t)(n + 1) * 2 * d);
  const size_t mx_b = al(sizeof(float) * ((size_t)P + 1));
  const size_t id_b = al(sizeof(uint32_t) * (size_t)(n + 1) * d);
  const size_t key_b = al(sizeof(uint32_t) * (size_t)n * d);
  const size_t bm_b = al(sizeof(float) * std::max<uint64_t>(1, (P + 1) >> kBlockLog));
  const size_t si_b = al(sizeof(uint32_t) * (size_t)((n + 63) / 64) * d);
  const size_t qu_b = al(sizeof(uint32_t) * kQuant * d);
  size_t strip_b = 0;
  if (d > 1) {
    const size_t slots = (size_t)strip_count(n) << kStripLog;
    strip_b = d * (al(sizeof(float) * slots * 2 * d) + al(sizeof(uint32_t) * slots) +
                   al(sizeof(float) * (slots / 64) * 2 * d));
  }
  return strip_b + al(sizeof(float) * (size_t)n * 2 * d) + rec_b * d + mx_b * d + id_b + 2 * key_b + bm_b * d + 2 * si_b + qu_b + 256 + 256 +
         al(sizeof(float) * 4 * DDM_MAX_D) + al(sizeof(uint32_t) * DDM_MAX_D * 2 * (kFeatBins + 1)) +
         al(sizeof(uint32_t) * kSatWords);
}

static TreeJobs make_jobs(const ddm_tree* t, const float* lo, const float* hi) {
  const bool sort_hi = t->d == 1;
  TreeJobs J{};
  for (uint32_t k = 0; k < t->d; ++k) {
    TreeJob& j = J.j[k];
    j.s_lo = lo;
    j.s_hi = hi;
    j.rec = t->rec[k];
    j.maxhi = t->maxhi[k];
    j.bmax = t->bmax[k];
    j.id = t->id[k];
    j.skey_lo = t->skey_lo[k];
    j.skey_hi = sort_hi ? t->skey_hi[k] : nullptr;
    j.sidx_lo = t->sidx_lo[k];
    j.sidx_hi = sort_hi ? t->sidx_hi[k] : nullptr;
    j.quant = t->quant[k];
    j.srec = t->srec[k];
    j.sid = t->sid[k];
    j.sbox = t->sbox[k];
    j.maxlen_bits = (uint32_t*)t->maxlen + k;
    j.n = t->n;
    j.d = t->d;
    j.k = k;
    j.P = t->P;
    j.C = t->C;
    j.H = t->H;
    j.ns = t->ns;
  }
  return J;
}

// the strips' dynamic LDS exceeds the default limit at d = 4
static ddm_status ensure_tree_attr() {
  static std::once_flag once;
  static hipError_t err = hipSuccess;
  std::call_once(once, [] {
    for (const void* f : {(const void*)tree_low_kernel, (const void*)tree_refit_kernel})
      if (err == hipSuccess)
        err = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)strip_lds_bytes(DDM_MAX_D));
  });
  if (err != hipSuccess) return hip_fail(err, "hipFuncSetAttribute", __FILE__, __LINE__);
  return DDM_OK;
}

// samples/quantiles of the sorted keys, maxupper and block maxima; the
// records are gathered from the inputs (gather) or already in place
static ddm_status enqueue_tree_passes(const ddm_tree* t, const TreeJobs& J, bool gather,
                                      hipStream_t s) {
  const uint32_t d = t->d;
  ProfScope ps("tree_build", s);
  const uint32_t ig = (std::max(t->ns, kQuant) + kTreeThreads - 1) / kTreeThreads;
  dim3 g((t->P + 1 + kChunk - 1) / kChunk + ig, d);
  const size_t lds = d > 1 ? strip_lds_bytes(d) : 0;
  if (lds) {
    const ddm_status st = ensure_tree_attr();
    if (st != DDM_OK) return st;
  }
  if (gather)
    tree_low_kernel<<<g, kTreeThreads, lds, s>>>(J, ig);
  else
    tree_refit_kernel<<<g, kTreeThreads, lds, s>>>(J, ig);
  DDM_LAUNCHED("tree_low_kernel");
  for (uint32_t S = kChunkLog; S < t->H; S += kChunkLog) {
    const uint32_t q_end = (t->P >> S) + 1;
    dim3 g2((q_end + kChunk - 1) / kChunk, d);
    tree_high_kernel<<<g2, kTreeThreads, 0, s>>>(J, S);
    DDM_LAUNCHED("tree_high_kernel");
  }
  return DDM_OK;
}

ddm_status enqueue_tree_build(ddm_tree* t, const float* lo, const float* hi, hipStream_t s) {
  const uint32_t n = t->n, d = t->d;
  // scratch: ping-pong key buffers (lo and hi), payload ping-pong, sort tables
  // upper bounds are sorted only for d == 1, where the BITS counts are the
  // final counts; for d > 1 the probe dimension comes from lower bounds only
  const bool sort_hi = d == 1;
  const uint32_t narr = sort_hi ? 2 * d : d;
  if (n <= kSmallMax) {
    {
      ProfScope ps("build_keys", s);
#define DDM_SMALL(R)                                                                     \
  build_small_kernel<R><<<narr, kSmallThreads, 0, s>>>(lo, hi, n, d, t->skey_lo[0],     \
                                                       t->skey_hi[0], t->id[0], t->flag, \
                                                       (uint32_t*)t->maxlen, t->rid)
      switch ((n + kSmallThreads - 1) / kSmallThreads) {
        case 1: DDM_SMALL(1); break;
        case 2: DDM_SMALL(2); break;
        case 3: DDM_SMALL(3); break;
        case 4: DDM_SMALL(4); break;
        case 5: DDM_SMALL(5); break;
        case 6: DDM_SMALL(6); break;
        default: DDM_SMALL(8); break;
      }
#undef DDM_SMALL
      DDM_LAUNCHED("build_small_kernel");
    }
    TreeJobs J = make_jobs(t, lo, hi);
    for (uint32_t k = 0; k < d; ++k) J.j[k].recin = t->rid;
    return enqueue_tree_passes(t, J, true, s);
  }
  // the sort's arrays (buffer 1 of each is filled in once scratch exists)
  SortArr host[2 * DDM_MAX_D];
  for (uint32_t i = 0; i < narr; ++i) host[i] = SortArr{{nullptr, nullptr}, {nullptr, nullptr}, n, 0};
  const size_t sort_bytes = radix_onesweep_scratch_bytes(host, narr, 4);
  Scratch sc(s);
  sc.reserve(sizeof(uint32_t) * (size_t)n * d);  // lo keys tmp
  sc.reserve(sizeof(uint32_t) * (size_t)n * d);  // hi keys tmp
  sc.reserve(sizeof(uint32_t) * (size_t)n * d);  // payload tmp
  sc.reserve(sort_bytes);
  if (!sc.commit()) return DDM_E_NOMEM;
  uint32_t* klo_tmp = sc.take<uint32_t>((size_t)n * d);
  uint32_t* khi_tmp = sc.take<uint32_t>((size_t)n * d);
  uint32_t* val_tmp = sc.take<uint32_t>((size_t)n * d);
  char* sort_scratch = sc.take<char>(sort_bytes);
  if (!sc.fits()) return scratch_overrun("tree build");

  uint32_t na = 0;
  for (uint32_t k = 0; k < d; ++k) {
    SortArr& a = host[na++];
    a.k[0] = t->skey_lo[k];
    a.k[1] = klo_tmp + (size_t)k * n;
    a.v[0] = t->id[k] + 1;
    a.v[1] = val_tmp + (size_t)k * n;
    if (!sort_hi) continue;
    SortArr& b = host[na++];
    b.k[0] = t->skey_hi[k];
    b.k[1] = khi_tmp + (size_t)k * n;
  }
  const OsScratch S = radix_onesweep_scratch(host, narr, 4, sort_scratch);
  {
    ProfScope ps("build_keys", s);
    const unsigned zb = (unsigned)std::min<size_t>((std::max<size_t>(S.nstatus, S.nhist) + 255) / 256, 2048);
    build_zero_kernel<<<zb, 256, 0, s>>>(t->flag, (uint32_t*)t->maxlen, d, S);
    DDM_LAUNCHED("build_zero_kernel");
    const unsigned g = (n + kKeyThreads * kKeyItems - 1) / (kKeyThreads * kKeyItems);
#define DDM_KEYS(DD)                                                                            \
  build_keys_kernel<DD><<<g, kKeyThreads, 0, s>>>(lo, hi, n, t->skey_lo[0],                     \
                                                  sort_hi ? t->skey_hi[0] : nullptr, t->id[0], \
                                                  t->flag, t->rid, S.ghist)
    switch (d) {
      case 1: DDM_KEYS(1); break;
      case 2: DDM_KEYS(2); break;
      case 3: DDM_KEYS(3); break;
      default: DDM_KEYS(4); break;
    }
#undef DDM_KEYS
    DDM_LAUNCHED("build_keys_kernel");
  }
  ddm_status st = radix_onesweep_passes(host, narr, 4, S, t->flag, s);
  if (st != DDM_OK) return st;
  TreeJobs J = make_jobs(t, lo, hi);
  for (uint32_t k = 0; k < d; ++k) J.j[k].recin = t->rid;
  return enqueue_tree_passes(t, J, true, s);
}

// ---------------------------------------------------------------------------
// Moving subscriptions of a resident tree (dynamic DDM: extents move between
// matches, Sec. I and Sec. VI).  If the moved lower bounds keep every tree's
// (lower bound, id) order, the records are rewritten in place and maxupper,
// block maxima, samples and quantiles are recomputed over the records
// (refit, no sort); otherwise the subscription set is read back from the
// records, the moves applied, and the tree rebuilt.
// ---------------------------------------------------------------------------
struct TreePtrs {
  float* rec[DDM_MAX_D];
  float* rid;  // records by id
  const uint32_t* id[DDM_MAX_D];
  uint32_t* pos[DDM_MAX_D];  // position of every subscription in tree k
  uint32_t* key[DDM_MAX_D];  // sorted lower keys with the moves applied
  uint32_t n, d;
};

__global__ void upd_pos_kernel(TreePtrs A) {
  const uint32_t k = blockIdx.y;
  const uint32_t p = 1 + blockIdx.x * blockDim.x + threadIdx.x;
  if (p <= A.n) A.pos[k][A.id[k][p]] = p;
}

// ids in range and new extents valid (flag bit 2)
__global__ void upd_check_kernel(const uint32_t* __restrict__ ids, const float* __restrict__ lo,
                                 const float* __restrict__ hi, uint32_t count, uint32_t n,
                                 uint32_t d, int32_t* __restrict__ flag) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  bool bad = ids[c] >= n;
  for (uint32_t k = 0; k < d; ++k)
    bad = bad || !valid_extent(lo[(size_t)k * count + c], hi[(size_t)k * count + c]);
  if (bad) atomicOr(flag, 4);
}

__global__ void upd_keys_kernel(TreePtrs A, const uint32_t* __restrict__ ids,
                                const float* __restrict__ lo, uint32_t count) {
  const uint32_t k = blockIdx.y;
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  const uint32_t i = ids[c];
  if (i >= A.n) return;
  A.key[k][A.pos[k][i] - 1] = f2key(lo[(size_t)k * count + c]);
}

// (key, id) strictly increasing along every tree after the moves? (bit 3)
__global__ void upd_order_kernel(TreePtrs A, int32_t* __restrict__ flag) {
  const uint32_t k = blockIdx.y;
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  bool bad = false;
  if (i + 1 < A.n) {
    const uint32_t a = A.key[k][i], b = A.key[k][i + 1];
    bad = a > b || (a == b && A.id[k][i + 1] > A.id[k][i + 2]);
  }
  // at most one atomic per workgroup, and none once the bit is seen: they queue
  // on the word (20,000 of 5*10^5 moved: 21 us, 48 without the look; 88 us with
  // one per entry and 5000 moved)
  if (__syncthreads_or(bad) && threadIdx.x == 0 &&
      !(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 8))
    atomicOr(flag, 8);
}

// the moved extents into their record of every tree
__global__ void upd_apply_kernel(TreePtrs A, const uint32_t* __restrict__ ids,
                                 const float* __restrict__ lo, const float* __restrict__ hi,
                                 uint32_t count) {
  const uint32_t k = blockIdx.y;
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  const uint32_t D = A.d;
  float* r = A.rec[k] + (size_t)A.pos[k][ids[c]] * 2 * D;
  r[0] = lo[(size_t)k * count + c];
  r[1] = hi[(size_t)k * count + c];
  A.rid[((size_t)ids[c] * D + k) * 2] = r[0];
  A.rid[((size_t)ids[c] * D + k) * 2 + 1] = r[1];
  uint32_t slot = 1;
  for (uint32_t kk = 0; kk < D; ++kk) {
    if (kk == k) continue;
    r[2 * slot] = lo[(size_t)kk * count + c];
    r[2 * slot + 1] = hi[(size_t)kk * count + c];
    ++slot;
  }
}

__global__ void upd_zero_maxlen_kernel(uint32_t* __restrict__ maxlen_bits, uint32_t d) {
  if (threadIdx.x < d) maxlen_bits[threadIdx.x] = 0;
}

// d = 1: upper keys of the records, to be sorted again
__global__ void upd_hi_keys_kernel(const float* __restrict__ rec, uint32_t n,
                                   uint32_t* __restrict__ khi) {
  const uint32_t p = 1 + blockIdx.x * blockDim.x + threadIdx.x;
  if (p <= n) khi[p - 1] = f2key(rec[(size_t)p * 2 + 1]);
}

// the subscription set back from tree 0's records (slot s holds dimension s)
__global__ void upd_gather_kernel(const float* __restrict__ rec, const uint32_t* __restrict__ id,
                                  uint32_t n, uint32_t d, float* __restrict__ lo,
                                  float* __restrict__ hi) {
  const uint32_t p = 1 + blockIdx.x * blockDim.x + threadIdx.x;
  if (p > n) return;
  const uint32_t i = id[p];
  const float* r = rec + (size_t)p * 2 * d;
  for (uint32_t k = 0; k < d; ++k) {
    lo[(size_t)k * n + i] = r[2 * k];
    hi[(size_t)k * n + i] = r[2 * k + 1];
  }
}

__global__ void upd_scatter_kernel(const uint32_t* __restrict__ ids,
                                   const float* __restrict__ nlo, const float* __restrict__ nhi,
                                   uint32_t count, uint32_t n, uint32_t d,
                                   float* __restrict__ lo, float* __restrict__ hi) {
  const uint32_t c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= count) return;
  const uint32_t i = ids[c];
  for (uint32_t k = 0; k < d; ++k) {
    lo[(size_t)k * n + i] = nlo[(size_t)k * count + c];
    hi[(size_t)k * n + i] = nhi[(size_t)k * count + c];
  }
}

static ddm_status tree_update(ddm_tree* t, const uint32_t* ids, const float* nlo,
                              const float* nhi, uint32_t count, hipStream_t s, int* rebuilt) {
  const uint32_t n = t->n, d = t->d;
  Scratch sc(s);
  sc.reserve(sizeof(uint32_t) * (size_t)n * d);  // positions
  sc.reserve(sizeof(uint32_t) * (size_t)n * d);  // keys with the moves
  sc.reserve(sizeof(int32_t));                   // flag
  if (!sc.commit()) return DDM_E_NOMEM;
  uint32_t* pos = sc.take<uint32_t>((size_t)n * d);
  uint32_t* keys = sc.take<uint32_t>((size_t)n * d);
  int32_t* flag = sc.take<int32_t>(1);
  if (!sc.fits()) return scratch_overrun("tree update");
  TreePtrs A{};
  for (uint32_t k = 0; k < d; ++k) {
    A.rec[k] = t->rec[k];
    A.id[k] = t->id[k];
    A.pos[k] = pos + (size_t)k * n;
    A.key[k] = keys + (size_t)k * n;
    DDM_HIP(hipMemcpyAsync(A.key[k], t->skey_lo[k], sizeof(uint32_t) * n,
                           hipMemcpyDeviceToDevice, s));
  }
  A.rid = t->rid;
  A.n = n;
  A.d = d;
  flag_zero_kernel<<<1, 64, 0, s>>>(flag);
  DDM_LAUNCHED("flag_zero_kernel");
  upd_pos_kernel<<<dim3((n + 255) / 256, d), 256, 0, s>>>(A);
  DDM_LAUNCHED("upd_pos_kernel");
  upd_check_kernel<<<(count + 255) / 256, 256, 0, s>>>(ids, nlo, nhi, count, n, d, flag);
  DDM_LAUNCHED("upd_check_kernel");
  upd_keys_kernel<<<dim3((count + 255) / 256, d), 256, 0, s>>>(A, ids, nlo, count);
  DDM_LAUNCHED("upd_keys_kernel");
  upd_order_kernel<<<dim3((n + 255) / 256, d), 256, 0, s>>>(A, flag);
  DDM_LAUNCHED("upd_order_kernel");
  int32_t f = 0;
  DDM_HIP(hipMemcpyAsync(&f, flag, sizeof(f), hipMemcpyDeviceToHost, s));
  DDM_HIP(hipStreamSynchronize(s));
  if (f & 4) {
    set_detail("ddm_tree_update: id out of range, or NaN/inf or lo > hi in the new extents");
    return DDM_E_INVALID_INPUT;
  }
  {
    // learned-sizing statistics describe the old set
    std::lock_guard<std::mutex> lk(t->fmu);
    t->fstats_ready = false;
  }
  if (!(f & 8)) {
    *rebuilt = 0;
    upd_apply_kernel<<<dim3((count + 255) / 256, d), 256, 0, s>>>(A, ids, nlo, nhi, count);
    DDM_LAUNCHED("upd_apply_kernel");
    for (uint32_t k = 0; k < d; ++k)
      DDM_HIP(hipMemcpyAsync(t->skey_lo[k], A.key[k], sizeof(uint32_t) * n,
                             hipMemcpyDeviceToDevice, s));
    upd_zero_maxlen_kernel<<<1, 64, 0, s>>>((uint32_t*)t->maxlen, d);
    DDM_LAUNCHED("upd_zero_maxlen_kernel");
    if (d == 1) {
      // the upper keys stay a sorted multiset for the exact counts
      SortArr h{{nullptr, nullptr}, {nullptr, nullptr}, n, 0};
      const size_t sort_bytes = radix_onesweep_scratch_bytes(&h, 1, 4);
      Scratch ss(s);
      ss.reserve(sizeof(uint32_t) * n);
      ss.reserve(sort_bytes);
      if (!ss.commit()) return DDM_E_NOMEM;
      uint32_t* ktmp = ss.take<uint32_t>(n);
      char* sort_scratch = ss.take<char>(sort_bytes);
      if (!ss.fits()) return scratch_overrun("tree update");
      upd_hi_keys_kernel<<<(n + 255) / 256, 256, 0, s>>>(t->rec[0], n, t->skey_hi[0]);
      DDM_LAUNCHED("upd_hi_keys_kernel");
      h.k[0] = t->skey_hi[0];
      h.k[1] = ktmp;
      ddm_status st = radix_sort_onesweep(&h, 1, 4, sort_scratch, t->flag, s);
      if (st != DDM_OK) return st;
      return enqueue_tree_passes(t, make_jobs(t, nullptr, nullptr), false, s);
    }
    return enqueue_tree_passes(t, make_jobs(t, nullptr, nullptr), false, s);
  }
  *rebuilt = 1;
  Scratch sr(s);
  sr.reserve(sizeof(float) * (size_t)n * d);
  sr.reserve(sizeof(float) * (size_t)n * d);
  if (!sr.commit()) return DDM_E_NOMEM;
  float* lo = sr.take<float>((size_t)n * d);
  float* hi = sr.take<float>((size_t)n * d);
  if (!sr.fits()) return scratch_overrun("tree update");
  upd_gather_kernel<<<(n + 255) / 256, 256, 0, s>>>(t->rec[0], t->id[0], n, d, lo, hi);
  DDM_LAUNCHED("upd_gather_kernel");
  upd_scatter_kernel<<<(count + 255) / 256, 256, 0, s>>>(ids, nlo, nhi, count, n, d, lo, hi);
  DDM_LAUNCHED("upd_scatter_kernel");
  return enqueue_tree_build(t, lo, hi, s);
}

// ---------------------------------------------------------------------------
// Few moves of a resident tree (d > 1): the sorted arrays stay sorted but for
// the moved entries, so every tree is merged instead of sorted again.  The
// moved entries are sorted by their old and by their new (key, id), one
// workgroup each; then every tile of old positions knows from three searches
// how many moved entries left and came before it, and every entry its new
// position.  The moved ids come in ascending order, distinct and checked.
// 5000 of 5*10^5 squares: 38 us in place of 84 us of keys and sort passes
// and 145 us for the order check and the set read back.
// ---------------------------------------------------------------------------
struct MoveArgs {
  const uint32_t* sid;  // c moved ids, ascending
  const float* lo;      // their new extents [d][c]
  const float* hi;
  const uint32_t* bits;        // the moved ids as a bitmap
  uint32_t* mkey[2 * DDM_MAX_D];  // array 2k: sorted old keys of dimension k, 2k + 1: new keys
  uint32_t* midx[2 * DDM_MAX_D];  // their places in sid
  uint32_t* key[DDM_MAX_D];    // the merged keys (0..n-1)
  uint32_t* id[DDM_MAX_D];     // and ids (positions 1..n)
  const uint32_t* okey[DDM_MAX_D];  // the tree's own
  const uint32_t* oid[DDM_MAX_D];
  float* rid;
  uint32_t* maxlen_bits;
  uint32_t c, n, d;
};

template <int R>
__global__ __launch_bounds__(kBlockSortThreads) void move_sort_kernel(MoveArgs A) {
  __shared__ BlockSortLds<R, uint16_t> L;
  const uint32_t k = blockIdx.x >> 1;
  const bool fresh = blockIdx.x & 1u;
  uint32_t id[R], key[R], val[R];
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = block_sort_index<R>(r);
    id[r] = i < A.c ? A.sid[i] : A.n;
  }
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = block_sort_index<R>(r);
    const bool ok = i < A.c && id[r] < A.n;  // (ids are only checked when the host has read the flag)
    const float v = !ok ? 0.f
                    : fresh ? A.lo[(size_t)k * A.c + i]
                            : A.rid[((size_t)id[r] * A.d + k) * 2];
    key[r] = f2key(v);
    val[r] = i;
  }
  block_sort<R>(L, key, val, A.c, 4);
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = block_sort_index<R>(r);
    if (i < A.c) {
      A.mkey[blockIdx.x][i] = key[r];
      A.midx[blockIdx.x][i] = val[r];
    }
  }
}

// moved entries (array a, sorted) below (x, id), by one wavefront
__device__ __forceinline__ uint32_t move_count_below(const MoveArgs& A, uint32_t a, uint32_t x,
                                                     uint32_t id) {
  uint32_t at = 0, len = A.c;
  while (len) {
    const uint32_t step = (len + kWave - 1) / kWave;
    const uint32_t o = lane_id() * step + step - 1;
    bool less = false;
    if (o < len) {
      const uint32_t y = A.mkey[a][at + o];
      less = y < x || (y == x && A.sid[A.midx[a][at + o]] < id);
    }
    const uint32_t full = (uint32_t)__popcll(ballot(less)) * step;
    at += full;
    len = min(step - 1, len - full);
  }
  return at;
}

constexpr uint32_t kMoveTile = 2048, kMoveThreads = 256, kMoveCache = 1024;

__global__ __launch_bounds__(kMoveThreads) void move_merge_kernel(MoveArgs A) {
  constexpr uint32_t R = kMoveTile / kMoveThreads, W = kMoveThreads / kWave;
  __shared__ uint32_t lk[kMoveTile], li[kMoveTile];
  __shared__ uint16_t gone[kMoveTile];  // moved entries before each, within the tile
  __shared__ uint32_t ck[kMoveCache], ci[kMoveCache];  // the entries that come into the tile
  __shared__ uint32_t wgone[R * W + 1];
  __shared__ uint32_t bound[3];
  const uint32_t k = blockIdx.y, tid = threadIdx.x, wave = tid / kWave, lane = lane_id();
  const uint32_t p0 = blockIdx.x * kMoveTile, tn = min(kMoveTile, A.n - p0);
  const uint32_t* __restrict__ okey = A.okey[k];
  const uint32_t* __restrict__ oid = A.oid[k] + 1;
  uint32_t key[R], id[R];
  bool mv[R];
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = r * kMoveThreads + tid;
    key[r] = i < tn ? okey[p0 + i] : 0u;
    id[r] = i < tn ? oid[p0 + i] : 0u;
  }
  // wavefront 0: moved entries whose old place is before the tile; 1: new
  // places before it; 2: new places before the next tile
  if (wave < 3) {
    const uint32_t at = wave < 2 ? p0 : p0 + kMoveTile;
    uint32_t v;
    if (at >= A.n)
      v = A.c;
    else if (at == 0)
      v = 0;
    else
      v = move_count_below(A, 2 * k + (wave ? 1u : 0u), okey[at], oid[at]);
    if (lane == 0) bound[wave] = v;
  }
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = r * kMoveThreads + tid;
    mv[r] = i < tn && ((A.bits[id[r] >> 5] >> (id[r] & 31u)) & 1u);
    lk[i] = key[r];
    li[i] = id[r];
    const uint64_t b = ballot(mv[r]);
    if (lane == 0) wgone[r * W + wave] = (uint32_t)__popcll(b);
  }
  __syncthreads();
  if (wave == 0) {
    const uint32_t v = lane < R * W ? wgone[lane] : 0u;
    const uint32_t inc = wave_scan_dpp(v);
    if (lane < R * W) wgone[lane] = inc - v;
    if (lane == R * W - 1) wgone[R * W] = inc;
  }
  const uint32_t o0 = bound[0], i0 = bound[1], i1 = bound[2];
  const uint32_t* __restrict__ nk = A.mkey[2 * k + 1];
  const uint32_t* __restrict__ ni = A.midx[2 * k + 1];
  const bool cached = i1 - i0 <= kMoveCache;
  if (cached)
    for (uint32_t q = i0 + tid; q < i1; q += kMoveThreads) {
      ck[q - i0] = nk[q];
      ci[q - i0] = A.sid[ni[q]];
    }
  __syncthreads();
#pragma unroll
  for (uint32_t r = 0; r < R; ++r) {
    const uint32_t i = r * kMoveThreads + tid;
    const uint32_t g = wgone[r * W + wave] + mask_rank(ballot(mv[r]));
    gone[i] = (uint16_t)g;
    if (i < tn && !mv[r]) {
      uint32_t at = i0, len = i1 - i0;
      while (len) {
        const uint32_t half = len >> 1, q = at + half;
        const uint32_t y = cached ? ck[q - i0] : nk[q];
        const bool less = y < key[r] ||
                          (y == key[r] && (cached ? ci[q - i0] : A.sid[ni[q]]) < id[r]);
        at = less ? q + 1 : at;
        len = less ? len - half - 1 : half;
      }
      const uint32_t dst = p0 + i - (o0 + g) + at;
      if (dst < A.n) {
        A.key[k][dst] = key[r];
        A.id[k][dst + 1] = id[r];
      }
    }
  }
  __syncthreads();
  for (uint32_t q = i0 + tid; q < i1; q += kMoveThreads) {
    const uint32_t x = nk[q], slot = ni[q], who = A.sid[slot];
    uint32_t at = 0, len = tn;
    while (len) {
      const uint32_t half = len >> 1, j = at + half;
      const bool less = lk[j] < x || (lk[j] == x && li[j] < who);
      at = less ? j + 1 : at;
      len = less ? len - half - 1 : half;
    }
    const uint32_t g = o0 + (at < tn ? (uint32_t)gone[at] : wgone[R * W]);
    const uint32_t dst = q + p0 + at - g;
    if (dst < A.n) {
      A.key[k][dst] = x;
      A.id[k][dst + 1] = who;
    }
    *reinterpret_cast<float2*>(A.rid + ((size_t)who * A.d + k) * 2) =
        make_float2(A.lo[(size_t)k * A.c + slot], A.hi[(size_t)k * A.c + slot]);
  }
  if (blockIdx.x == 0 && tid == 0) A.maxlen_bits[k] = 0;
}

bool tree_move_ok(const ddm_tree* t, uint32_t count) {
  return t->d > 1 && count <= kTreeMoveMax && count <= t->n;
}

size_t tree_move_words(const ddm_tree* t, uint32_t count) {
  return 4 * (size_t)t->d * count + t->d * (2 * (size_t)t->n + 1);
}

static MoveArgs move_args(const ddm_tree* t, const TreeMove& M) {
  MoveArgs A{};
  A.sid = M.sid;
  A.lo = M.lo;
  A.hi = M.hi;
  A.bits = M.bits;
  A.c = M.count;
  A.n = t->n;
  A.d = t->d;
  A.rid = t->rid;
  A.maxlen_bits = (uint32_t*)t->maxlen;
  uint32_t* p = M.words;
  for (uint32_t a = 0; a < 2 * t->d; ++a) {
    A.mkey[a] = p;
    A.midx[a] = p + M.count;
    p += 2 * (size_t)M.count;
  }
  for (uint32_t k = 0; k < t->d; ++k) {
    A.key[k] = p;
    A.id[k] = p + t->n;
    p += 2 * (size_t)t->n + 1;
    A.okey[k] = t->skey_lo[k];
    A.oid[k] = t->id[k];
  }
  return A;
}

ddm_status tree_move_sort(const ddm_tree* t, const TreeMove& M, hipStream_t s) {
  static_assert(kTreeMoveMax <= 8 * kBlockSortThreads, "the largest sort");
  const MoveArgs A = move_args(t, M);
#define DDM_MOVE(R) move_sort_kernel<R><<<2 * t->d, kBlockSortThreads, 0, s>>>(A)
  switch ((M.count + kBlockSortThreads - 1) / kBlockSortThreads) {
    case 1: DDM_MOVE(1); break;
    case 2: DDM_MOVE(2); break;
    case 3: DDM_MOVE(3); break;
    case 4: DDM_MOVE(4); break;
    case 5: DDM_MOVE(5); break;
    case 6: DDM_MOVE(6); break;
    default: DDM_MOVE(8); break;
  }
#undef DDM_MOVE
  DDM_LAUNCHED("move_sort_kernel");
  return DDM_OK;
}

ddm_status tree_move_apply(ddm_tree* t, const TreeMove& M, hipStream_t s) {
  const MoveArgs A = move_args(t, M);
  {
    // learned-sizing statistics describe the old set
    std::lock_guard<std::mutex> lk(t->fmu);
    t->fstats_ready = false;
  }
  move_merge_kernel<<<dim3((t->n + kMoveTile - 1) / kMoveTile, t->d), kMoveThreads, 0, s>>>(A);
  DDM_LAUNCHED("move_merge_kernel");
  TreeJobs J = make_jobs(t, nullptr, nullptr);
  for (uint32_t k = 0; k < t->d; ++k) {
    J.j[k].recin = t->rid;
    J.j[k].id = A.id[k];
    J.j[k].skey_lo = A.key[k];
    J.j[k].id_out = t->id[k];
    J.j[k].key_out = t->skey_lo[k];
  }
  return enqueue_tree_passes(t, J, true, s);
}

// Enqueue the feature statistics on stream s the first time a learned match
// uses the tree; later users on other streams wait for the recorded event.
ddm_status tree_ensure_features(const ddm_tree* tc, hipStream_t s) {
  ddm_tree* t = const_cast<ddm_tree*>(tc);
  std::lock_guard<std::mutex> lk(t->fmu);
  if (t->fstats_ready) {
    DDM_HIP(hipStreamWaitEvent(s, t->fstats_event, 0));
    return DDM_OK;
  }
  ProfScope ps("feature_stats", s);
  FeatArgs F{};
  for (uint32_t k = 0; k < t->d; ++k) {
    F.rec[k] = t->rec[k];
    F.maxhi[k] = t->maxhi[k];
    F.skey_lo[k] = t->skey_lo[k];
    F.sidx_lo[k] = t->sidx_lo[k];
  }
  F.n = t->n;
  F.d = t->d;
  F.ns = t->ns;
  F.root = 1u << (t->H - 1);
  F.fstat = t->fstat;
  F.fcum = t->fcum;
  F.sat = t->sat;
  ddm_status st = enqueue_feature_stats(F, s);
  if (st != DDM_OK) return st;
  if (!t->fstats_event) t->fstats_event = pooled_event();
  if (!t->fstats_event) {
    set_detail("event creation failed");
    return DDM_E_DEVICE;
  }
  DDM_HIP(hipEventRecord(t->fstats_event, s));
  t->fstats_ready = true;
  return DDM_OK;
}

}  // namespace ddm

using namespace ddm;

extern "C" ddm_status ddm_build(const float* sub_lo, const float* sub_hi, uint32_t n, uint32_t d,
                                void* stream, ddm_tree** out_tree) {
  set_detail("");
  if (!out_tree) {
    set_detail("ddm_build: out_tree is NULL");
    return DDM_E_INVALID_ARG;
  }
  *out_tree = nullptr;
  if (d < 1 || d > DDM_MAX_D) {
    set_detail("ddm_build: d must be in [1, DDM_MAX_D]");
    return DDM_E_INVALID_ARG;
  }
  if (n > 0 && (!sub_lo || !sub_hi)) {
    set_detail("ddm_build: NULL coordinate pointer");
    return DDM_E_INVALID_ARG;
  }
  if (n >= 0x40000000u) {
    set_detail("ddm_build: n must be below 2^30");
    return DDM_E_INVALID_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  ddm_tree* t = new (std::nothrow) ddm_tree();
  if (!t) return DDM_E_NOMEM;
  DDM_HIP(hipGetDevice(&t->device));
  t->stream = s;
  t->n = n;
  t->d = d;
  if (n == 0) {
    *out_tree = t;
    return DDM_OK;
  }
  uint32_t H = 0;
  while (H < 32 && ((1ull << H) - 1) < n) ++H;
  t->H = H;
  t->P = (uint32_t)((1ull << H) - 1);
  const size_t rec_b = al(sizeof(float) * (size_t)(n + 1) * 2 * d);
  const size_t mx_b = al(sizeof(float) * ((size_t)t->P + 1));
  const size_t id_b = al(sizeof(uint32_t) * (size_t)(n + 1) * d);
  const size_t key_b = al(sizeof(uint32_t) * (size_t)n * d);
  t->C = std::max<uint32_t>(1u, (uint32_t)(((uint64_t)t->P + 1) >> kBlockLog));
  const size_t bm_b = al(sizeof(float) * t->C);
  t->ns = (n + 63) / 64;
  const size_t si_b = al(sizeof(uint32_t) * (size_t)t->ns * d);
  const size_t qu_b = al(sizeof(uint32_t) * kQuant * d);
  const size_t total = tree_bytes_estimate(n, d);
  void* blk = dev_alloc(total, s);
  if (!blk) {
    delete t;
    set_detail("ddm_build: device allocation failed");
    return DDM_E_NOMEM;
  }
  t->block = (char*)blk;
  char* p = t->block;
  for (uint32_t k = 0; k < d; ++k) { t->rec[k] = (float*)p; p += rec_b; }
  for (uint32_t k = 0; k < d; ++k) { t->maxhi[k] = (float*)p; p += mx_b; }
  uint32_t* idb = (uint32_t*)p;
  p += id_b;
  for (uint32_t k = 0; k < d; ++k) t->id[k] = idb + (size_t)k * (n + 1);
  uint32_t* klo = (uint32_t*)p;
  p += key_b;
  uint32_t* khi = (uint32_t*)p;
  p += key_b;
  for (uint32_t k = 0; k < d; ++k) {
    t->skey_lo[k] = klo + (size_t)k * n;
    t->skey_hi[k] = khi + (size_t)k * n;
  }
  for (uint32_t k = 0; k < d; ++k) { t->bmax[k] = (float*)p; p += bm_b; }
  {
    uint32_t* ilo = (uint32_t*)p;
    p += si_b;
    uint32_t* ihi = (uint32_t*)p;
    p += si_b;
    for (uint32_t k = 0; k < d; ++k) {
      t->sidx_lo[k] = ilo + (size_t)k * t->ns;
      t->sidx_hi[k] = ihi + (size_t)k * t->ns;
    }
    uint32_t* qu = (uint32_t*)p;
    p += qu_b;
    for (uint32_t k = 0; k < d; ++k) t->quant[k] = qu + (size_t)k * kQuant;
  }
  if (d > 1) {
    const size_t slots = (size_t)strip_count(n) << kStripLog;
    for (uint32_t k = 0; k < d; ++k) {
      t->srec[k] = (float*)p;
      p += al(sizeof(float) * slots * 2 * d);
      t->sid[k] = (uint32_t*)p;
      p += al(sizeof(uint32_t) * slots);
      t->sbox[k] = (float*)p;
      p += al(sizeof(float) * (slots / 64) * 2 * d);
    }
  }
  t->rid = (float*)p;
  p += al(sizeof(float) * (size_t)n * 2 * d);
  t->maxlen = (float*)p;
  p += 256;
  t->fstat = (float*)p;
  p += al(sizeof(float) * 4 * DDM_MAX_D);
  t->fcum = (uint32_t*)p;
  p += al(sizeof(uint32_t) * DDM_MAX_D * 2 * (kFeatBins + 1));
  t->sat = (uint32_t*)p;
  p += al(sizeof(uint32_t) * kSatWords);
  t->flag = (int32_t*)p;
  ddm_status st = enqueue_tree_build(t, sub_lo, sub_hi, s);
  if (st != DDM_OK) {
    dev_free(t->block, s);
    delete t;
    return st;
  }
  *out_tree = t;
  return DDM_OK;
}

extern "C" ddm_status ddm_tree_update(ddm_tree* t, const uint32_t* ids, const float* new_lo,
                                      const float* new_hi, uint32_t count, void* stream,
                                      int* out_rebuilt) {
  set_detail("");
  if (!t || (count && (!ids || !new_lo || !new_hi))) {
    set_detail("ddm_tree_update: NULL argument");
    return DDM_E_INVALID_ARG;
  }
  if (out_rebuilt) *out_rebuilt = 0;
  if (count == 0) return DDM_OK;
  if (t->n == 0 || count > t->n) {
    set_detail("ddm_tree_update: more moves than subscriptions");
    return DDM_E_INVALID_ARG;
  }
  int cur = -1;
  DDM_HIP(hipGetDevice(&cur));
  if (cur != t->device) {
    set_detail("ddm_tree_update: the current device is not the tree's device");
    return DDM_E_INVALID_ARG;
  }
  int rb = 0;
  ddm_status st = tree_update(t, ids, new_lo, new_hi, count, (hipStream_t)stream, &rb);
  if (out_rebuilt) *out_rebuilt = rb;
  return st;
}

extern "C" void ddm_tree_free(ddm_tree* t) {
  if (!t) return;
  release_event(t->fstats_event);
  if (t->block) {
    int cur = 0;
    (void)hipGetDevice(&cur);
    if (cur != t->device) (void)hipSetDevice(t->device);
    dev_free(t->block, t->stream);
    if (cur != t->device) (void)hipSetDevice(cur);
  }
  delete t;
}

extern "C" ddm_status ddm_tree_check(const ddm_tree* t) {
  set_detail("");
  if (!t) return DDM_E_INVALID_ARG;
  if (t->n == 0) return DDM_OK;
  int32_t f = 0;
  DDM_HIP(hipStreamSynchronize(t->stream));
  DDM_HIP(hipMemcpy(&f, t->flag, sizeof(f), hipMemcpyDeviceToHost));
  if (f & kFlagSortTimeout) {
    set_detail("tree build: a radix sort look-back wait gave up");
    return DDM_E_DEVICE;
  }
  if (f) {
    set_detail("subscription coordinates: NaN/inf or lo > hi");
    return DDM_E_INVALID_INPUT;
  }
  return DDM_OK;
}

extern "C" ddm_status ddm_tree_prepare_learned(const ddm_tree* t, void* stream) {
  set_detail("");
  if (!t) return DDM_E_INVALID_ARG;
  if (t->d > 3) {
    set_detail("features are defined for d <= 3");
    return DDM_E_INVALID_ARG;
  }
  if (t->n == 0) {
    set_detail("features need a non-empty subscription set");
    return DDM_E_INVALID_ARG;
  }
  return tree_ensure_features(t, (hipStream_t)stream);
}

extern "C" ddm_status ddm_tree_info(const ddm_tree* t, uint32_t* n, uint32_t* d, uint32_t* height) {
  if (!t) return DDM_E_INVALID_ARG;
  if (n) *n = t->n;
  if (d) *d = t->d;
  if (height) *height = t->H;
  return DDM_OK;
}

extern "C" ddm_status ddm_tree_export(const ddm_tree* t, uint32_t k, float* lo, float* hi,
                                      uint32_t* ids, float* maxhi) {
  set_detail("");
  if (!t || k >= t->d) return DDM_E_INVALID_ARG;
  if (t->n == 0) return DDM_OK;
  DDM_HIP(hipStreamSynchronize(t->stream));
  const uint32_t n = t->n, D = t->d;
  if (lo || hi) {
    float* recs = (float*)malloc(sizeof(float) * (size_t)(n + 1) * 2 * D);
    if (!recs) return DDM_E_NOMEM;
    hipError_t e = hipMemcpy(recs, t->rec[k], sizeof(float) * (size_t)(n + 1) * 2 * D,
                             hipMemcpyDeviceToHost);
    if (e != hipSuccess) {
      free(recs);
      return hip_fail(e, "hipMemcpy", __FILE__, __LINE__);
    }
    for (uint32_t p = 1; p <= n; ++p) {
      if (lo) lo[p - 1] = recs[(size_t)p * 2 * D];
      if (hi) hi[p - 1] = recs[(size_t)p * 2 * D + 1];
    }
    free(recs);
  }
  if (ids) DDM_HIP(hipMemcpy(ids, t->id[k] + 1, sizeof(uint32_t) * n, hipMemcpyDeviceToHost));
  if (maxhi)
    DDM_HIP(hipMemcpy(maxhi, t->maxhi[k] + 1, sizeof(float) * t->P, hipMemcpyDeviceToHost));
  return DDM_OK;
}
