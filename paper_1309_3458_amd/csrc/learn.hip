// Learned output sizing: a small MLP (18 -> 64 -> 64 -> 1, FP32, ReLU) that
// predicts log1p(number of subscriptions an update meets) from the update's
// extent and coarse prefix histograms of the subscription endpoints.  It
// only sizes the output of the single-pass matcher; every pair still comes
// from the exact traversal, and an update whose prediction falls short is
// redone by the plain count -> scan -> fill path, so results never depend on
// the network.
//
// Kernels: per-tree feature statistics (built with the tree), per-update
// features, forward (inference and capacities), forward + backward with
// per-workgroup partial gradients reduced in a fixed order (deterministic),
// and Adam.
#include "ddm_internal.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

namespace ddm {

// ---------------------------------------------------------------------------
// parameter layout (row-major W[out][in])
// ---------------------------------------------------------------------------
constexpr int kIn = kFeatures;
constexpr int kHid = 64;
constexpr int oW1 = 0;
constexpr int oB1 = oW1 + kHid * kIn;    // 1152
constexpr int oW2 = oB1 + kHid;          // 1216
constexpr int oB2 = oW2 + kHid * kHid;   // 5312
constexpr int oW3 = oB2 + kHid;          // 5376
constexpr int oB3 = oW3 + kHid;          // 5440
static_assert(oB3 + 1 == kParams, "parameter count");

// ---------------------------------------------------------------------------
// per-tree feature statistics (enqueued by the tree build)
//   fstat[k] = {min lower bound, width = max upper - min lower, mean length}
//   fcum[k][0][b] = #{lo < e_b}, fcum[k][1][b] = #{hi in bins < b},
//   e_b = min + width * b / 64, b = 0..64
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t hist_bin(float x, float mn, float w) {
  const float u = (x - mn) / w * (float)kFeatBins;
  if (!(u > 0.f)) return 0u;
  return min((uint32_t)u, (uint32_t)kFeatBins - 1u);
}

__global__ __launch_bounds__(256) void feat_hist_kernel(FeatArgs A, double* __restrict__ part) {
  __shared__ uint32_t h[kFeatBins];
  __shared__ double ws[256 / kWave];
  const uint32_t k = blockIdx.y;
  const uint32_t D = A.d;
  const uint32_t tid = threadIdx.x;
  if (tid < kFeatBins) h[tid] = 0;
  __syncthreads();
  const float mn = A.rec[k][2 * D];  // lower bound at in-order position 1
  const float mx = A.maxhi[k][A.root];
  const float w = fmaxf(mx - mn, 1e-30f);
  double ext = 0.0;
  for (uint32_t p = 1 + blockIdx.x * 256 + tid; p <= A.n; p += gridDim.x * 256) {
    const float lo = A.rec[k][(size_t)p * 2 * D];
    const float hi = A.rec[k][(size_t)p * 2 * D + 1];
    atomicAdd(&h[hist_bin(hi, mn, w)], 1u);
    ext += (double)hi - (double)lo;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) ext += __shfl_xor(ext, o, kWave);
  if (lane_id() == 0) ws[tid / kWave] = ext;
  __syncthreads();
  if (tid < kFeatBins && h[tid]) atomicAdd(&A.fcum[(k * 2 + 1) * (kFeatBins + 1) + tid + 1], h[tid]);
  if (tid == 0) {
    double t = 0.0;
    for (int i = 0; i < 256 / kWave; ++i) t += ws[i];
    part[(size_t)k * gridDim.x + blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(128) void feat_final_kernel(FeatArgs A, const double* __restrict__ part,
                                                         uint32_t nparts) {
  const uint32_t k = blockIdx.x;
  const uint32_t D = A.d;
  const float mn = A.rec[k][2 * D];
  const float mx = A.maxhi[k][A.root];
  const float w = fmaxf(mx - mn, 1e-30f);
  const uint32_t b = threadIdx.x;
  if (b <= kFeatBins) {
    const float e = (b == kFeatBins) ? mx : mn + w * (float)b / (float)kFeatBins;
    const uint32_t* keys[1] = {A.skey_lo[k]};
    const uint32_t* idx[1] = {A.sidx_lo[k]};
    const uint32_t x[1] = {f2key(e)};
    const bool up[1] = {b == kFeatBins};
    uint32_t res[1];
    count_2l<1>(keys, idx, x, up, A.n, A.ns, res);
    A.fcum[(k * 2) * (kFeatBins + 1) + b] = res[0];
  }
  __syncthreads();
  if (b == 0) {
    uint32_t* c = A.fcum + (k * 2 + 1) * (kFeatBins + 1);
    c[0] = 0;
    for (uint32_t i = 1; i <= (uint32_t)kFeatBins; ++i) c[i] += c[i - 1];
    double t = 0.0;
    for (uint32_t i = 0; i < nparts; ++i) t += part[(size_t)k * nparts + i];
    A.fstat[k * 4 + 0] = mn;
    A.fstat[k * 4 + 1] = w;
    A.fstat[k * 4 + 2] = (float)(t / (double)A.n);
    A.fstat[k * 4 + 3] = 0.f;
  }
}

__global__ void feat_zero_kernel(uint32_t* __restrict__ fcum, uint32_t count,
                                 uint32_t* __restrict__ sat) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) fcum[i] = 0;
  if (i < kSatWords) sat[i] = 0;
}

// joint histogram of the subscriptions' lower corners on a G^d grid over the
// bounding box; entry (i0+1, i1+1, ...) of the (G+1)^d array counts the
// corners of cell (i0, i1, ...).  Corners are read from tree 0's records
// (lower bound of dimension 0, then those of the other dimensions).  Each
// workgroup counts into LDS and adds its nonzero cells to the global array.
__global__ __launch_bounds__(256) void sat_hist_kernel(FeatArgs A) {
  __shared__ uint32_t h[kSatWords];
  const uint32_t D = A.d;
  if (D > 3) return;
  const uint32_t G = sat_grid(D);
  uint32_t cells = 1;
  for (uint32_t k = 0; k < D; ++k) cells *= G + 1;
  for (uint32_t i = threadIdx.x; i < cells; i += 256) h[i] = 0;
  __syncthreads();
  for (uint32_t p = 1 + blockIdx.x * 256 + threadIdx.x; p <= A.n; p += gridDim.x * 256) {
    uint32_t idx = 0, stride = 1;
    for (uint32_t k = 0; k < D; ++k) {
      const float lo = A.rec[0][(size_t)p * 2 * D + 2 * k];
      const float u = (lo - A.fstat[k * 4 + 0]) / A.fstat[k * 4 + 1] * (float)G;
      const uint32_t c = !(u > 0.f) ? 0u : min((uint32_t)u, G - 1u);
      idx += (c + 1) * stride;
      stride *= G + 1;
    }
    atomicAdd(&h[idx], 1u);
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < cells; i += 256)
    if (h[i]) atomicAdd(&A.sat[i], h[i]);
}

// prefix sums along every axis in LDS: sat[i...] = corners in cells < i
__global__ __launch_bounds__(1024) void sat_prefix_kernel(FeatArgs A) {
  __shared__ uint32_t h[kSatWords];
  const uint32_t D = A.d;
  if (D > 3) return;
  const uint32_t G1 = sat_grid(D) + 1;
  uint32_t cells = 1;
  for (uint32_t k = 0; k < D; ++k) cells *= G1;
  for (uint32_t i = threadIdx.x; i < cells; i += blockDim.x) h[i] = A.sat[i];
  __syncthreads();
  const uint32_t lines = cells / G1;
  uint32_t stride = 1;
  for (uint32_t ax = 0; ax < D; ++ax) {
    for (uint32_t l = threadIdx.x; l < lines; l += blockDim.x) {
      // base index: l enumerates the other axes
      uint32_t base = 0, rem = l, st = 1;
      for (uint32_t k = 0; k < D; ++k) {
        if (k != ax) {
          base += (rem % G1) * st;
          rem /= G1;
        }
        st *= G1;
      }
      uint32_t run = 0;
      for (uint32_t i = 0; i < G1; ++i) {
        run += h[base + i * stride];
        h[base + i * stride] = run;
      }
    }
    stride *= G1;
    __syncthreads();
  }
  for (uint32_t i = threadIdx.x; i < cells; i += blockDim.x) A.sat[i] = h[i];
}

ddm_status enqueue_feature_stats(const FeatArgs& A, hipStream_t s) {
  const uint32_t nparts = 64;
  Scratch sc(s);
  sc.reserve(sizeof(double) * nparts * A.d);
  if (!sc.commit()) return DDM_E_NOMEM;
  double* part = sc.take<double>(nparts * A.d);
  if (!sc.fits()) return scratch_overrun("feature statistics");
  const uint32_t cnt = A.d * 2 * (kFeatBins + 1);
  feat_zero_kernel<<<(std::max(cnt, kSatWords) + 255) / 256, 256, 0, s>>>(A.fcum, cnt, A.sat);
  DDM_LAUNCHED("feat_zero_kernel");
  feat_hist_kernel<<<dim3(nparts, A.d), 256, 0, s>>>(A, part);
  DDM_LAUNCHED("feat_hist_kernel");
  feat_final_kernel<<<A.d, 128, 0, s>>>(A, part, nparts);
  DDM_LAUNCHED("feat_final_kernel");
  if (A.d <= 3) {
    sat_hist_kernel<<<nparts, 256, 0, s>>>(A);
    DDM_LAUNCHED("sat_hist_kernel");
    sat_prefix_kernel<<<1, 1024, 0, s>>>(A);
    DDM_LAUNCHED("sat_prefix_kernel");
  }
  return DDM_OK;
}

// ---------------------------------------------------------------------------
// features of one update (d <= 3), see the header for their definition
// ---------------------------------------------------------------------------
__device__ __forceinline__ float interp_cum(const uint32_t* __restrict__ c, float u) {
  if (!(u > 0.f)) return (float)c[0];
  if (u >= (float)kFeatBins) return (float)c[kFeatBins];
  const uint32_t b = (uint32_t)u;
  const float fr = u - (float)b;
  return (float)c[b] + fr * ((float)c[b + 1] - (float)c[b]);
}

// corners counted by the prefix array below the point u (grid units, one per
// dimension), multilinear inside a cell (corners spread evenly in a cell).
// Evaluated in double: the box count below is a signed sum of 2^d such
// values that can cancel to a small number.
template <int D>
__device__ __forceinline__ double sat_at(const uint32_t* __restrict__ sat, const float (&u)[D]) {
  constexpr uint32_t G = sat_grid(D);
  uint32_t i[D];
  double f[D];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const float uk = fminf(fmaxf(u[k], 0.f), (float)G);
    i[k] = min((uint32_t)uk, G - 1u);
    f[k] = (double)uk - (double)i[k];
  }
  double acc = 0.0;
#pragma unroll
  for (int c = 0; c < (1 << D); ++c) {
    double w = 1.0;
    uint32_t idx = 0, st = 1;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const bool hi = (c >> k) & 1;
      w *= hi ? f[k] : 1.0 - f[k];
      idx += (i[k] + (hi ? 1u : 0u)) * st;
      st *= G + 1;
    }
    acc += w * (double)sat[idx];
  }
  return acc;
}

// corners in the box [a, b] (grid units), by inclusion-exclusion
template <int D>
__device__ __forceinline__ double sat_box(const uint32_t* __restrict__ sat, const float (&a)[D],
                                          const float (&b)[D]) {
  double tot = 0.0;
#pragma unroll
  for (int c = 0; c < (1 << D); ++c) {
    float u[D];
    int neg = 0;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      const bool hi = (c >> k) & 1;
      u[k] = hi ? b[k] : a[k];
      neg += hi ? 0 : 1;
    }
    const double v = sat_at<D>(sat, u);
    tot += (neg & 1) ? -v : v;
  }
  return tot;
}

template <int D>
__global__ __launch_bounds__(256) void features_kernel(FeatDev F, const float* __restrict__ ulo,
                                                       const float* __restrict__ uhi, uint32_t m,
                                                       float* __restrict__ X) {
  const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= m) return;
  float f[kFeatures];
#pragma unroll
  for (int i = 0; i < kFeatures; ++i) f[i] = 0.f;
  const float n = (float)F.n;
  constexpr float G = (float)sat_grid(D);
  float ga[D], gb[D];
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const float ql = ulo[(size_t)k * m + j], qh = uhi[(size_t)k * m + j];
    const float mn = F.fstat[k * 4 + 0], w = F.fstat[k * 4 + 1], me = F.fstat[k * 4 + 2];
    const uint32_t* clo = F.fcum + (k * 2) * (kFeatBins + 1);
    const uint32_t* chi = F.fcum + (k * 2 + 1) * (kFeatBins + 1);
    const float c_le = interp_cum(clo, (qh - mn) / w * (float)kFeatBins);
    const float c_lt = interp_cum(chi, (ql - mn) / w * (float)kFeatBins);
    const float c = fminf(fmaxf(c_le - c_lt, 0.f), n);
    f[5 * k + 0] = (qh - ql) / w;
    f[5 * k + 1] = (0.5f * (ql + qh) - mn) / w;
    f[5 * k + 2] = c / n;
    f[5 * k + 3] = log1pf(c) * (1.f / 16.f);
    f[5 * k + 4] = me / w;
    // lower corners that can meet q in this dimension: [q.lo - mean length, q.hi]
    ga[k] = (ql - me - mn) / w * G;
    gb[k] = (qh - mn) / w * G;
  }
  f[15] = log2f(n) * (1.f / 20.f);
  f[16] = (float)D * (1.f / 3.f);
  f[17] = log1pf((float)fmax(sat_box<D>(F.sat, ga, gb), 0.0)) * (1.f / 16.f);
#pragma unroll
  for (int i = 0; i < kFeatures; ++i) X[(size_t)j * kFeatures + i] = f[i];
}

ddm_status launch_features(const FeatDev& F, uint32_t d, const float* ulo, const float* uhi,
                           uint32_t m, float* X, hipStream_t s) {
  if (m == 0) return DDM_OK;
  ProfScope ps("features", s);
  switch (d) {
    case 1: features_kernel<1><<<(m + 255) / 256, 256, 0, s>>>(F, ulo, uhi, m, X); break;
    case 2: features_kernel<2><<<(m + 255) / 256, 256, 0, s>>>(F, ulo, uhi, m, X); break;
    case 3: features_kernel<3><<<(m + 255) / 256, 256, 0, s>>>(F, ulo, uhi, m, X); break;
    default:
      set_detail("features: d must be at most 3");
      return DDM_E_INVALID_ARG;
  }
  DDM_LAUNCHED("features_kernel");
  return DDM_OK;
}

// ---------------------------------------------------------------------------
// The network on the matrix cores (v_mfma_f32_16x16x4_f32: FP32 products and
// sums).  A wavefront takes 16 samples; a layer is out = W in, with the
// outputs as rows and the samples as columns of the product, so that lane l
// holds, for sample l % 16, the outputs 16t + 4(l/16) + r of tile t (r < 4).
// The contraction of the next layer may run over its inputs in any order as
// long as both operands use the same one: step (t, r) takes input
// 16t + 4(l/16) + r in lane l, which is the register the lane already holds,
// so the activations never leave their lanes.  The weights are the other
// operand, kept in registers over all of a wavefront's samples.
// Bound by the matrix unit: 84 products of 32 cycles per 16 samples forward,
// 244 for the gradient.
// ---------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kMT = kHid / 16;        // row tiles of a hidden layer
constexpr int kInSteps = 5;           // ceil(kIn / 4) contraction steps of the first layer
static_assert(kIn <= 4 * kInSteps - 1, "a spare input column holds the bias gradient's ones");

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 load_f32x4(const float* p) {
  f32x4 v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = p[r];
  return v;
}

struct MlpRegs {
  float w1[kMT][kInSteps];  // W1[16t + l%16][4s + l/16], 0 past kIn
  f32x4 w2[kMT][kMT];       // W2[16t + l%16][16u + 4(l/16) + r]
  f32x4 b1[kMT], b2[kMT], w3[kMT];
  float b3;
};

__device__ __forceinline__ void mlp_load(const float* __restrict__ P, MlpRegs& W) {
  const int c = (int)(lane_id() & 15u), q = (int)(lane_id() >> 4);
#pragma unroll
  for (int t = 0; t < kMT; ++t) {
#pragma unroll
    for (int s = 0; s < kInSteps; ++s) {
      const int i = 4 * s + q;
      W.w1[t][s] = i < kIn ? P[oW1 + (16 * t + c) * kIn + i] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kMT; ++u) W.w2[t][u] = load_f32x4(P + oW2 + (16 * t + c) * kHid + 16 * u + 4 * q);
    W.b1[t] = load_f32x4(P + oB1 + 16 * t + 4 * q);
    W.b2[t] = load_f32x4(P + oB2 + 16 * t + 4 * q);
    W.w3[t] = load_f32x4(P + oW3 + 16 * t + 4 * q);
  }
  W.b3 = P[oB3];
}

// x[s] = input 4s + l/16 of sample l % 16; returns the prediction of sample
// l % 16 (in every lane of that sample)
__device__ __forceinline__ float mlp_eval(const MlpRegs& W, const float (&x)[kInSteps],
                                          f32x4 (&h1)[kMT], f32x4 (&h2)[kMT]) {
#pragma unroll
  for (int t = 0; t < kMT; ++t) h1[t] = W.b1[t];
#pragma unroll
  for (int s = 0; s < kInSteps; ++s)
#pragma unroll
    for (int t = 0; t < kMT; ++t) h1[t] = mfma4(W.w1[t][s], x[s], h1[t]);
#pragma unroll
  for (int t = 0; t < kMT; ++t) {
#pragma unroll
    for (int r = 0; r < 4; ++r) h1[t][r] = fmaxf(h1[t][r], 0.f);
    h2[t] = W.b2[t];
  }
#pragma unroll
  for (int u = 0; u < kMT; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int t = 0; t < kMT; ++t) h2[t] = mfma4(W.w2[t][u][r], h1[u][r], h2[t]);
  float y = 0.f;
#pragma unroll
  for (int t = 0; t < kMT; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h2[t][r] = fmaxf(h2[t][r], 0.f);
      y = fmaf(W.w3[t][r], h2[t][r], y);
    }
  y += __shfl_xor(y, 16, kWave);
  y += __shfl_xor(y, 32, kWave);
  return y + W.b3;
}

// ---------------------------------------------------------------------------
// MLP forward
//   out_mode 0: yhat[s] = prediction
//   out_mode 1: cap[s] = min(ceil(expm1(prediction + delta)), capmax)
// One thread per sample with the parameters in LDS took 26.7 us for 4096
// samples and 102 us for 5*10^5; this form 5.6 and 57.
// ---------------------------------------------------------------------------
constexpr int kFwdWaves = 4;

__global__ __launch_bounds__(kFwdWaves * kWave) void mlp_forward_kernel(
    const float* __restrict__ params, const float* __restrict__ X, uint32_t N, int out_mode,
    float delta, uint32_t capmax, float* __restrict__ yhat, uint32_t* __restrict__ cap) {
  MlpRegs W;
  mlp_load(params, W);
  const uint32_t lane = lane_id(), c = lane & 15u, q = lane >> 4;
  const uint32_t wave = blockIdx.x * kFwdWaves + threadIdx.x / kWave;
  const uint32_t nw = gridDim.x * kFwdWaves;
  const uint32_t tiles = (N + 15u) / 16u;
  for (uint32_t tl = wave; tl < tiles; tl += nw) {
    const uint32_t sidx = tl * 16u + c;
    float x[kInSteps];
#pragma unroll
    for (uint32_t s = 0; s < kInSteps; ++s) {
      const uint32_t i = 4u * s + q;
      x[s] = sidx < N && i < (uint32_t)kIn ? X[(size_t)sidx * kIn + i] : 0.f;
    }
    f32x4 h1[kMT], h2[kMT];
    const float y = mlp_eval(W, x, h1, h2);
    if (q != 0 || sidx >= N) continue;
    if (out_mode == 0) {
      yhat[sidx] = y;
    } else {
      const float e = expm1f(fminf(y + delta, 30.f));
      const float v = ceilf(fmaxf(e, 0.f));
      cap[sidx] = v >= (float)capmax ? capmax : (uint32_t)v;
    }
  }
}

ddm_status launch_mlp_forward(const float* params, const float* X, uint32_t N, int out_mode,
                              float delta, uint32_t capmax, float* yhat, uint32_t* cap,
                              hipStream_t s) {
  if (N == 0) return DDM_OK;
  ProfScope ps("mlp_forward", s);
  // one 16-sample tile per wavefront up to 8 wavefronts per compute unit,
  // then several tiles for each set of weights loaded
  const uint32_t blocks = std::min<uint32_t>((N + 16 * kFwdWaves - 1) / (16 * kFwdWaves), 512);
  mlp_forward_kernel<<<blocks, kFwdWaves * kWave, 0, s>>>(params, X, N, out_mode, delta, capmax,
                                                         yhat, cap);
  DDM_LAUNCHED("mlp_forward_kernel");
  return DDM_OK;
}

// ---------------------------------------------------------------------------
// MLP forward + backward of the mean squared error over N samples.
// A wavefront runs 16 samples forward and back (dz2 as computed, dz1 = W2^T
// dz2 with the activations' lane layout again), turns h1, dz2, dy h2 and dz1
// through LDS to put the samples on the contraction, and adds dW2 = dz2 h1^T
// and dW1 = dz1 [x, 1]^T to accumulators it keeps over all its samples.  The
// workgroup's wavefronts then add up in a fixed order, one partial gradient
// per workgroup; mlp_reduce_kernel sums the partials in a fixed order.
// One thread per sample, 128 samples per workgroup, took 87 us for 4096
// samples (32 workgroups on 256 compute units); this form 27.
// ---------------------------------------------------------------------------
constexpr int kGradWaves = 4;
constexpr int kGradBlocks = 256;  // at most: partials of one gradient
constexpr int kTS = 80;           // LDS row of a sample: 16 lanes x 4 rows hit 64 banks once

__global__ __launch_bounds__(kGradWaves * kWave) void mlp_grad_kernel(
    const float* __restrict__ params, const float* __restrict__ X, const float* __restrict__ Y,
    uint32_t N, float* __restrict__ part, float* __restrict__ part_loss) {
  __shared__ float sH[kGradWaves][16 * kTS];  // h1, by sample
  __shared__ float sD[kGradWaves][16 * kTS];  // dz2
  __shared__ float sG[kGradWaves][16 * kTS];  // dy h2, then dz1
  __shared__ float acc[kParams];
  __shared__ float sloss[kGradWaves];
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = tid / kWave;
  const uint32_t c = lane & 15u, q = lane >> 4;
  float* H = sH[w];
  float* D = sD[w];
  float* G = sG[w];
  MlpRegs W;
  mlp_load(params, W);
  const float invN = 1.f / (float)N;
  f32x4 g2[kMT][kMT], g1[kMT][2];  // dW2[16t + ..][16u + ..], dW1 (column kIn: db1)
#pragma unroll
  for (int t = 0; t < kMT; ++t) {
#pragma unroll
    for (int u = 0; u < kMT; ++u) g2[t][u] = f32x4{0.f, 0.f, 0.f, 0.f};
    g1[t][0] = g1[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float gb2 = 0.f, gw3 = 0.f;  // db2, dW3 of output `lane`
  float gb3 = 0.f, loss = 0.f;
  const uint32_t tiles = (N + 15u) / 16u;
  for (uint32_t tl = blockIdx.x * kGradWaves + w; tl < tiles; tl += gridDim.x * kGradWaves) {
    const uint32_t s0 = tl * 16u, sidx = s0 + c;
    const bool valid = sidx < N;
    float x[kInSteps];
#pragma unroll
    for (uint32_t s = 0; s < kInSteps; ++s) {
      const uint32_t i = 4u * s + q;
      x[s] = valid && i < (uint32_t)kIn ? X[(size_t)sidx * kIn + i] : 0.f;
    }
    // [x, 1, 0 ..] with the samples on the contraction: column 16v + c of
    // sample 4s + q
    float xt[2][4];
#pragma unroll
    for (uint32_t v = 0; v < 2; ++v)
#pragma unroll
      for (uint32_t s = 0; s < 4; ++s) {
        const uint32_t si = s0 + 4u * s + q, i = 16u * v + c;
        xt[v][s] = si >= N ? 0.f
                   : i < (uint32_t)kIn ? X[(size_t)si * kIn + i]
                                       : (i == (uint32_t)kIn ? 1.f : 0.f);
      }
    const float ylab = valid ? Y[sidx] : 0.f;
    f32x4 h1[kMT], h2[kMT], d2[kMT], d1[kMT];
    const float y = mlp_eval(W, x, h1, h2);
    const float r = valid ? (y - ylab) : 0.f;
    const float dy = 2.f * r * invN;
    if (q == 0) {
      gb3 += dy;
      loss = fmaf(r * invN, r, loss);
    }
#pragma unroll
    for (int t = 0; t < kMT; ++t) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        d2[t][k] = h2[t][k] > 0.f ? dy * W.w3[t][k] : 0.f;
        const uint32_t at = c * kTS + 16u * t + 4u * q + k;
        H[at] = h1[t][k];
        D[at] = d2[t][k];
        G[at] = dy * h2[t][k];
      }
      d1[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // dz1 = W2^T dz2, masked (weights W2[16u + 4q + k][16t + c], cached)
#pragma unroll
    for (int u = 0; u < kMT; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int t = 0; t < kMT; ++t)
          d1[t] = mfma4(params[oW2 + (16 * u + 4 * (int)q + k) * kHid + 16 * t + (int)c], d2[u][k],
                        d1[t]);
#pragma unroll
    for (int t = 0; t < kMT; ++t)
#pragma unroll
      for (int k = 0; k < 4; ++k) d1[t][k] = h1[t][k] > 0.f ? d1[t][k] : 0.f;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      gb2 += D[s * kTS + lane];
      gw3 += G[s * kTS + lane];
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      float a[kMT], b[kMT];
#pragma unroll
      for (int t = 0; t < kMT; ++t) {
        a[t] = D[(4 * s + q) * kTS + 16 * t + c];
        b[t] = H[(4 * s + q) * kTS + 16 * t + c];
      }
#pragma unroll
      for (int t = 0; t < kMT; ++t)
#pragma unroll
        for (int u = 0; u < kMT; ++u) g2[t][u] = mfma4(a[t], b[u], g2[t][u]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int t = 0; t < kMT; ++t)
#pragma unroll
      for (int k = 0; k < 4; ++k) G[c * kTS + 16u * t + 4u * q + k] = d1[t][k];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int t = 0; t < kMT; ++t) {
        const float a = G[(4 * s + q) * kTS + 16 * t + c];
        g1[t][0] = mfma4(a, xt[0][s], g1[t][0]);
        g1[t][1] = mfma4(a, xt[1][s], g1[t][1]);
      }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    gb3 += __shfl_xor(gb3, o, kWave);
    loss += __shfl_xor(loss, o, kWave);
  }
  if (lane == 0) sloss[w] = loss;
  // the wavefronts add their gradients one after the other
  for (uint32_t v = 0; v < (uint32_t)kGradWaves; ++v) {
    if (w == v) {
      auto put = [&](uint32_t at, float val) { acc[at] = v == 0 ? val : acc[at] + val; };
#pragma unroll
      for (int t = 0; t < kMT; ++t)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const uint32_t o = 16u * t + 4u * q + k;
#pragma unroll
          for (int u = 0; u < kMT; ++u) put(oW2 + o * kHid + 16u * u + c, g2[t][u][k]);
          put(oW1 + o * kIn + c, g1[t][0][k]);
          if (16u + c < (uint32_t)kIn) put(oW1 + o * kIn + 16u + c, g1[t][1][k]);
          if (16u + c == (uint32_t)kIn) put(oB1 + o, g1[t][1][k]);
        }
      put(oB2 + lane, gb2);
      put(oW3 + lane, gw3);
      if (lane == 0) put(oB3, gb3);
    }
    __syncthreads();
  }
  float* g = part + (size_t)blockIdx.x * kParams;
  for (uint32_t i = tid; i < (uint32_t)kParams; i += kGradWaves * kWave) g[i] = acc[i];
  if (tid == 0) {
    float l = 0.f;
    for (int v = 0; v < kGradWaves; ++v) l += sloss[v];
    part_loss[blockIdx.x] = l;
  }
}

// 64 parameters per workgroup; wavefront g adds the partials g, g + 4, ..
// (their loads in flight together), then the four sums add up
constexpr uint32_t kRedGroups = 4;

__global__ __launch_bounds__(kRedGroups * kWave) void mlp_reduce_kernel(
    const float* __restrict__ part, const float* __restrict__ part_loss, uint32_t nb,
    float* __restrict__ grad, float* __restrict__ loss) {
  __shared__ float s[kRedGroups][kWave];
  const uint32_t lane = lane_id(), g = threadIdx.x / kWave;
  const uint32_t p = blockIdx.x * kWave + lane;
  float a = 0.f;
  if (p < (uint32_t)kParams) {
#pragma unroll 8
    for (uint32_t b = g; b < nb; b += kRedGroups) a += part[(size_t)b * kParams + p];
  }
  s[g][lane] = a;
  __syncthreads();
  if (g == 0 && p < (uint32_t)kParams) {
    for (uint32_t v = 1; v < kRedGroups; ++v) a += s[v][lane];
    grad[p] = a;
  }
  if (g == 1 && blockIdx.x == 0 && loss) {
    float l = 0.f;
    for (uint32_t b = lane; b < nb; b += kWave) l += part_loss[b];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o, kWave);
    if (lane == 0) *loss = l;
  }
}

ddm_status launch_mlp_grad(const float* params, const float* X, const float* Y, uint32_t N,
                           float* grad, float* loss, hipStream_t s) {
  if (N == 0) {
    set_detail("mlp gradient of an empty batch");
    return DDM_E_INVALID_ARG;
  }
  const uint32_t nb =
      std::min<uint32_t>((N + 16 * kGradWaves - 1) / (16 * kGradWaves), kGradBlocks);
  Scratch sc(s);
  sc.reserve(sizeof(float) * kParams * (size_t)nb);
  sc.reserve(sizeof(float) * nb);
  if (!sc.commit()) return DDM_E_NOMEM;
  float* part = sc.take<float>(kParams * (size_t)nb);
  float* pl = sc.take<float>(nb);
  if (!sc.fits()) return scratch_overrun("predictor gradient");
  ProfScope ps("mlp_grad", s);
  mlp_grad_kernel<<<nb, kGradWaves * kWave, 0, s>>>(params, X, Y, N, part, pl);
  DDM_LAUNCHED("mlp_grad_kernel");
  mlp_reduce_kernel<<<(kParams + kWave - 1) / kWave, kRedGroups * kWave, 0, s>>>(part, pl, nb,
                                                                              grad, loss);
  DDM_LAUNCHED("mlp_reduce_kernel");
  return DDM_OK;
}

__global__ void adam_kernel(float* __restrict__ params, float* __restrict__ m1,
                            float* __restrict__ m2, const float* __restrict__ grad, float lr,
                            float b1, float b2, float eps, float c1, float c2) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (uint32_t)kParams) return;
  const float g = grad[p];
  const float a = b1 * m1[p] + (1.f - b1) * g;
  const float v = b2 * m2[p] + (1.f - b2) * g * g;
  m1[p] = a;
  m2[p] = v;
  params[p] -= lr * (a / c1) / (sqrtf(v / c2) + eps);
}

// counter-based uniform numbers for the initial weights (splitmix64)
__device__ __forceinline__ float init_uniform(uint64_t seed, uint64_t i) {
  uint64_t z = seed + (i + 1) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z ^= z >> 31;
  return (float)(z >> 40) * (1.f / 16777216.f);
}

// U(-1/sqrt(fan_in), 1/sqrt(fan_in)) for weights and biases of each layer
__global__ void mlp_init_kernel(float* __restrict__ params, uint64_t seed) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= (uint32_t)kParams) return;
  const float fan = p < (uint32_t)oW2 ? (float)kIn : (p < (uint32_t)oW3 ? (float)kHid : (float)kHid);
  const float bound = 1.f / sqrtf(fan);
  params[p] = (2.f * init_uniform(seed, p) - 1.f) * bound;
}

__global__ void fill_f32_kernel(float* __restrict__ p, float v, uint32_t count) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

}  // namespace ddm

using namespace ddm;

struct ddm_predictor {
  int device = 0;
  float* block = nullptr;  // params | adam m | adam v | grad | loss
  float* params = nullptr;
  float* m1 = nullptr;
  float* m2 = nullptr;
  float* grad = nullptr;
  float* loss = nullptr;
  uint64_t step = 0;
  float delta = 0.f;
};

namespace ddm {
const float* predictor_params(const ddm_predictor* p) { return p->params; }
float predictor_delta(const ddm_predictor* p) { return p->delta; }
int predictor_device(const ddm_predictor* p) { return p->device; }
}  // namespace ddm

extern "C" ddm_status ddm_predictor_create(uint64_t seed, ddm_predictor** out) {
  set_detail("");
  if (!out) return DDM_E_INVALID_ARG;
  *out = nullptr;
  ddm_predictor* p = new (std::nothrow) ddm_predictor();
  if (!p) return DDM_E_NOMEM;
  DDM_HIP(hipGetDevice(&p->device));
  const size_t words = (size_t)kParams * 4 + 64;
  hipError_t e = hipMalloc((void**)&p->block, words * sizeof(float));
  if (e != hipSuccess) {
    delete p;
    (void)hipGetLastError();
    set_detail("predictor allocation failed");
    return DDM_E_NOMEM;
  }
  p->params = p->block;
  p->m1 = p->params + kParams;
  p->m2 = p->m1 + kParams;
  p->grad = p->m2 + kParams;
  p->loss = p->grad + kParams;
  mlp_init_kernel<<<(kParams + 255) / 256, 256>>>(p->params, seed);
  fill_f32_kernel<<<(2 * kParams + 255) / 256, 256>>>(p->m1, 0.f, 2 * kParams);
  e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    (void)hipFree(p->block);
    delete p;
    return hip_fail(e, "ddm_predictor_create", __FILE__, __LINE__);
  }
  *out = p;
  return DDM_OK;
}

extern "C" void ddm_predictor_free(ddm_predictor* p) {
  if (!p) return;
  if (p->block) (void)hipFree(p->block);
  delete p;
}

extern "C" ddm_status ddm_predictor_get_params(const ddm_predictor* p, float* host,
                                               uint32_t count, float* delta) {
  set_detail("");
  if (!p || (count && !host)) return DDM_E_INVALID_ARG;
  if (count != 0 && count != (uint32_t)kParams) {
    set_detail("count must be DDM_PREDICTOR_PARAMS");
    return DDM_E_INVALID_ARG;
  }
  if (count) DDM_HIP(hipMemcpy(host, p->params, sizeof(float) * kParams, hipMemcpyDeviceToHost));
  if (delta) *delta = p->delta;
  return DDM_OK;
}

extern "C" ddm_status ddm_predictor_set_params(ddm_predictor* p, const float* host,
                                               uint32_t count, float delta) {
  set_detail("");
  if (!p || (count && !host)) return DDM_E_INVALID_ARG;
  if (count != 0 && count != (uint32_t)kParams) {
    set_detail("count must be DDM_PREDICTOR_PARAMS");
    return DDM_E_INVALID_ARG;
  }
  if (!std::isfinite(delta)) {
    set_detail("delta must be finite");
    return DDM_E_INVALID_ARG;
  }
  if (count) {
    for (uint32_t i = 0; i < count; ++i)
      if (!std::isfinite(host[i])) {
        set_detail("parameters must be finite");
        return DDM_E_INVALID_ARG;
      }
    DDM_HIP(hipMemcpy(p->params, host, sizeof(float) * kParams, hipMemcpyHostToDevice));
  }
  p->delta = delta;
  return DDM_OK;
}

// Predictor file: "DDMP", format version, parameter count, delta (as its
// float bits), each a little-endian 32-bit word, then the parameters.
static const char kPredMagic[4] = {'D', 'D', 'M', 'P'};
constexpr uint32_t kPredVersion = 1;

extern "C" ddm_status ddm_predictor_save(const ddm_predictor* p, const char* path) {
  set_detail("");
  if (!p || !path) return DDM_E_INVALID_ARG;
  std::vector<float> w(kParams);
  float delta = 0.f;
  ddm_status st = ddm_predictor_get_params(p, w.data(), (uint32_t)kParams, &delta);
  if (st != DDM_OK) return st;
  uint32_t hdr[4];
  std::memcpy(&hdr[0], kPredMagic, 4);
  hdr[1] = kPredVersion;
  hdr[2] = (uint32_t)kParams;
  std::memcpy(&hdr[3], &delta, 4);
  FILE* f = std::fopen(path, "wb");
  if (!f) {
    set_detail(std::string("ddm_predictor_save: cannot open ") + path);
    return DDM_E_INVALID_ARG;
  }
  const bool ok = std::fwrite(hdr, sizeof(hdr), 1, f) == 1 &&
                  std::fwrite(w.data(), sizeof(float), w.size(), f) == w.size();
  if (std::fclose(f) != 0 || !ok) {
    set_detail(std::string("ddm_predictor_save: write failed: ") + path);
    return DDM_E_INVALID_ARG;
  }
  return DDM_OK;
}

extern "C" ddm_status ddm_predictor_load(const char* path, ddm_predictor** out) {
  set_detail("");
  if (!path || !out) return DDM_E_INVALID_ARG;
  *out = nullptr;
  FILE* f = std::fopen(path, "rb");
  if (!f) {
    set_detail(std::string("ddm_predictor_load: cannot open ") + path);
    return DDM_E_INVALID_ARG;
  }
  uint32_t hdr[4];
  std::vector<float> w(kParams);
  bool ok = std::fread(hdr, sizeof(hdr), 1, f) == 1 && std::memcmp(&hdr[0], kPredMagic, 4) == 0 &&
            hdr[1] == kPredVersion && hdr[2] == (uint32_t)kParams &&
            std::fread(w.data(), sizeof(float), w.size(), f) == w.size();
  char extra;
  ok = ok && std::fread(&extra, 1, 1, f) == 0;  // nothing after the parameters
  std::fclose(f);
  if (!ok) {
    set_detail(std::string("ddm_predictor_load: not a predictor file of this version: ") + path);
    return DDM_E_INVALID_INPUT;
  }
  float delta;
  std::memcpy(&delta, &hdr[3], 4);
  ddm_predictor* p = nullptr;
  ddm_status st = ddm_predictor_create(0, &p);
  if (st != DDM_OK) return st;
  st = ddm_predictor_set_params(p, w.data(), (uint32_t)kParams, delta);
  if (st != DDM_OK) {
    const std::string why = ddm_last_error_detail();
    ddm_predictor_free(p);
    set_detail("ddm_predictor_load: " + why);
    return DDM_E_INVALID_INPUT;
  }
  *out = p;
  return DDM_OK;
}

extern "C" ddm_status ddm_predictor_forward(const ddm_predictor* p, const float* X, uint32_t N,
                                            float* yhat, void* stream) {
  set_detail("");
  if (!p || (N && (!X || !yhat))) return DDM_E_INVALID_ARG;
  return launch_mlp_forward(p->params, X, N, 0, 0.f, 0, yhat, nullptr, (hipStream_t)stream);
}

extern "C" ddm_status ddm_predictor_grad(const ddm_predictor* p, const float* X, const float* Y,
                                         uint32_t N, float* grad, float* loss, void* stream) {
  set_detail("");
  if (!p || !X || !Y || !grad || N == 0) return DDM_E_INVALID_ARG;
  return launch_mlp_grad(p->params, X, Y, N, grad, loss, (hipStream_t)stream);
}

extern "C" ddm_status ddm_predictor_adam(ddm_predictor* p, const float* grad, float lr,
                                         void* stream) {
  set_detail("");
  if (!p || !grad || !(lr > 0.f)) return DDM_E_INVALID_ARG;
  const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
  p->step += 1;
  const float c1 = 1.f - (float)std::pow((double)b1, (double)p->step);
  const float c2 = 1.f - (float)std::pow((double)b2, (double)p->step);
  adam_kernel<<<(kParams + 255) / 256, 256, 0, (hipStream_t)stream>>>(p->params, p->m1, p->m2,
                                                                     grad, lr, b1, b2, eps, c1, c2);
  DDM_LAUNCHED("adam_kernel");
  return DDM_OK;
}

extern "C" ddm_status ddm_predictor_train(ddm_predictor* p, const float* X, const float* Y,
                                          uint32_t N, uint32_t batch, uint32_t epochs, float lr,
                                          void* stream, float* epoch_loss) {
  set_detail("");
  if (!p || !X || !Y || N == 0 || batch == 0 || epochs == 0 || !(lr > 0.f))
    return DDM_E_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const uint32_t nbat = (N + batch - 1) / batch;
  Scratch sc(s);
  sc.reserve(sizeof(float) * (size_t)nbat * epochs);
  if (!sc.commit()) return DDM_E_NOMEM;
  float* losses = sc.take<float>((size_t)nbat * epochs);
  if (!sc.fits()) return scratch_overrun("predictor training");
  for (uint32_t e = 0; e < epochs; ++e) {
    for (uint32_t b = 0; b < nbat; ++b) {
      const uint32_t s0 = b * batch;
      const uint32_t nb = std::min(batch, N - s0);
      ddm_status r = launch_mlp_grad(p->params, X + (size_t)s0 * kIn, Y + s0, nb, p->grad,
                                     losses + (size_t)e * nbat + b, s);
      if (r != DDM_OK) return r;
      r = ddm_predictor_adam(p, p->grad, lr, stream);
      if (r != DDM_OK) return r;
    }
  }
  if (epoch_loss) {
    std::vector<float> h((size_t)nbat * epochs);
    DDM_HIP(hipMemcpyAsync(h.data(), losses, sizeof(float) * h.size(), hipMemcpyDeviceToHost, s));
    DDM_HIP(hipStreamSynchronize(s));
    for (uint32_t e = 0; e < epochs; ++e) {
      double t = 0.0, w = 0.0;
      for (uint32_t b = 0; b < nbat; ++b) {
        const double nb = std::min(batch, N - b * batch);
        t += h[(size_t)e * nbat + b] * nb;
        w += nb;
      }
      epoch_loss[e] = (float)(t / w);
    }
  }
  return DDM_OK;
}
