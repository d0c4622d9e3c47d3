// Gaussian-hill bias on the device, FP64: evaluation of V and dV/ds, and the
// deposition of one well-tempered hill.  Fixed-order sums (thread -> wave ->
// block -> last block over the block partials), so results are reproducible.
#include "gm_device.h"

namespace gm {

// --------------------------------------------------------------------------
// Gaussian-hill bias (FP64): evaluation, or deposition of one hill.
// --------------------------------------------------------------------------
// s - c, or its nearest periodic image for a periodic dimension.
__device__ __forceinline__ double cv_delta(double s, double c, double period) {
  const double x = s - c;
  return period > 0.0 ? x - period * rint(x / period) : x;
}

// Fixed-order block sums of N values at once, valid in thread 0: wave sums, then
// the first wave adds the waves' sums.  All threads call; lds holds N kBiasBlock /
// 64 doubles and is free again when the block passes its next barrier.
template <int N>
__device__ __forceinline__ void block_sums(double (&v)[N], double (*lds)[3]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, waves = (int)(blockDim.x >> 6);
#pragma unroll
  for (int q = 0; q < N; q++) {
    v[q] = wave_sum(v[q]);
    if (lane == 0) lds[w][q] = v[q];
  }
  __syncthreads();
  if (w == 0)
#pragma unroll
    for (int q = 0; q < N; q++) {
      v[q] = lane < waves ? lds[lane][q] : 0.0;
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) v[q] += __shfl_down(v[q], o, 64);
    }
}

// V and dV/ds (v: V, then dV/ds), or the deposit of one hill (thread 0, once per
// evaluation).
template <int DIMS>
__device__ __forceinline__ void bias_result(const BiasArgs& a, int64_t K, const double (&v)[1 + DIMS]) {
  if (!isfinite(v[0])) atomicOr(a.err, kErrNonFinite);
  if (a.deposit) {
    const double h = a.wt_scale == 0.0 ? a.w0 : a.w0 * exp(-v[0] * a.wt_scale);
    if (K < a.capacity) {
      for (int d = 0; d < DIMS; d++) a.centres[K * DIMS + d] = a.s[d];
      a.heights[K] = h;
      *a.count = K + 1;
    } else {
      atomicOr(a.err, kErrCapacity);
    }
  } else {
    if (a.V_out) a.V_out[0] = v[0];
    if (a.dV_out)
      for (int d = 0; d < DIMS; d++) a.dV_out[d] = v[1 + d];
  }
}

// The sum over the hills.  One workgroup of 1,024 threads sums up to kBiasOne
// hills and is done; more hills are shared by workgroups whose partial sums a
// second launch adds in their order.  Latency bounds both (replayed from a graph):
// 4,000 hills 4.7 us in one launch and 5.4 in two (2-D: 5.6 and 6.2), 6,000 hills
// 6.6 and 5.4 (7.7 and 6.3).  A last-to-finish workgroup that adds the partials
// in the same launch takes longer than the second launch (7.8 us and 6.4).
template <int DIMS>
__device__ __forceinline__ void bias_sum(const BiasArgs& a, int32_t blk, int32_t nblk) {
  static_assert(kBiasBlock / 64 <= 16, "block_sums adds 16 waves");
  __shared__ double red[kBiasBlock / 64][3];
  const int64_t K = *a.count;
  double s[DIMS], v[1 + DIMS] = {};
#pragma unroll
  for (int d = 0; d < DIMS; d++) s[d] = a.s[d];
  auto add = [&](const double (&c)[DIMS], double h) {
    double x[DIMS], arg = 0.0;
#pragma unroll
    for (int d = 0; d < DIMS; d++) {
      x[d] = cv_delta(s[d], c[d], a.period[d]);
      arg += x[d] * x[d] * a.inv2s2[d];
    }
    const double e = h * exp(-arg);
    v[0] += e;
#pragma unroll
    for (int d = 0; d < DIMS; d++) v[1 + d] -= e * x[d] * a.invs2[d];
  };
  if (nblk == 1) {
    // up to 4 hills per thread and round, loaded as one batch (the last hill in
    // the place of those past the end, which are not added)
    for (int64_t k0 = threadIdx.x; k0 < K; k0 += 4 * kBiasBlock) {
      double c[4][DIMS], h[4];
#pragma unroll
      for (int u = 0; u < 4; u++) {
        const int64_t k = k0 + u * kBiasBlock < K ? k0 + u * kBiasBlock : K - 1;
#pragma unroll
        for (int d = 0; d < DIMS; d++) c[u][d] = a.centres[k * DIMS + d];
        h[u] = a.heights[k];
      }
#pragma unroll
      for (int u = 0; u < 4; u++)
        if (k0 + u * kBiasBlock < K) add(c[u], h[u]);
    }
  } else {
    // kBlock threads each, however many a batched launch gives them
    const int64_t stride = (int64_t)nblk * kBlock;
    for (int64_t k = threadIdx.x < kBlock ? (int64_t)blk * kBlock + threadIdx.x : K; k < K; k += stride) {
      double c[DIMS];
#pragma unroll
      for (int d = 0; d < DIMS; d++) c[d] = a.centres[k * DIMS + d];
      add(c, a.heights[k]);
    }
  }
  block_sums(v, red);
  if (threadIdx.x != 0) return;
  if (nblk == 1) {
    bias_result<DIMS>(a, K, v);
  } else {
#pragma unroll
    for (int q = 0; q <= DIMS; q++) a.part[blk * 3 + q] = v[q];
  }
}

__device__ __forceinline__ void bias_body(const BiasArgs& a, int32_t blk, int32_t nblk) {
  if (a.dims > 1)
    bias_sum<2>(a, blk, nblk);
  else
    bias_sum<1>(a, blk, nblk);
}

// Fixed-order sum of the partials of an evaluation by more than one workgroup.
template <int DIMS>
__device__ __forceinline__ void bias_finish_sum(const BiasArgs& a, int32_t nblk) {
  __shared__ double red[kBlock / 64][3];
  const int64_t K = *a.count;
  double v[1 + DIMS] = {};
  for (int32_t i = threadIdx.x; i < nblk; i += blockDim.x)
#pragma unroll
    for (int q = 0; q <= DIMS; q++) v[q] += a.part[i * 3 + q];
  block_sums(v, red);
  if (threadIdx.x == 0) bias_result<DIMS>(a, K, v);
}

__device__ __forceinline__ void bias_finish_body(const BiasArgs& a, int32_t nblk) {
  if (nblk == 1) return;
  if (a.dims > 1)
    bias_finish_sum<2>(a, nblk);
  else
    bias_finish_sum<1>(a, nblk);
}

__global__ __launch_bounds__(kBiasBlock) void k_bias(BiasArgs a) { bias_body(a, blockIdx.x, gridDim.x); }

__global__ __launch_bounds__(kBlock) void k_bias_finish(BiasArgs a, int32_t nblk) { bias_finish_body(a, nblk); }

__global__ __launch_bounds__(kBlock) void k_bias_finish_batch(const BiasArgs* __restrict__ tab,
                                                              const int32_t* __restrict__ blk_start) {
  const int32_t w = blockIdx.x;
  bias_finish_body(tab[w], blk_start[w + 1] - blk_start[w]);
}

// One launch for many walkers: workgroup g serves walker w with
// blk_start[w] <= g < blk_start[w+1].
__global__ __launch_bounds__(kBiasBlock) void k_bias_batch(const BiasArgs* __restrict__ tab,
                                                           const int32_t* __restrict__ blk_start, int32_t W) {
  const int64_t g = blockIdx.x;
  int32_t lo = 0, hi = W;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (blk_start[mid] <= g) lo = mid; else hi = mid;
  }
  bias_body(tab[lo], (int32_t)(g - blk_start[lo]), blk_start[lo + 1] - blk_start[lo]);
}

hipError_t launch_bias_batch(const BiasArgs* tab, const int32_t* blk_start, int32_t W, int32_t blocks,
                             hipStream_t st) {
  k_bias_batch<<<(unsigned)blocks, kBiasBlock, 0, st>>>(tab, blk_start, W);
  if (blocks > W) k_bias_finish_batch<<<(unsigned)W, kBlock, 0, st>>>(tab, blk_start);
  return hipGetLastError();
}

// The same for a subset of a batch's walkers named by value.
__global__ __launch_bounds__(kBiasBlock) void k_bias_subset(BiasSubset s) {
  const int32_t g = blockIdx.x;
  int32_t lo = 0, hi = s.k;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (s.blk[mid] <= g) lo = mid; else hi = mid;
  }
  bias_body(*s.tab[lo], g - s.blk[lo], s.blk[lo + 1] - s.blk[lo]);
}

__global__ __launch_bounds__(kBlock) void k_bias_finish_subset(BiasSubset s) {
  const int32_t w = blockIdx.x;
  bias_finish_body(*s.tab[w], s.blk[w + 1] - s.blk[w]);
}

hipError_t launch_bias_subset(const BiasSubset& s, hipStream_t st) {
  if (s.k < 1) return hipSuccess;
  k_bias_subset<<<(unsigned)s.blk[s.k], kBiasBlock, 0, st>>>(s);
  if (s.blk[s.k] > s.k) k_bias_finish_subset<<<(unsigned)s.k, kBlock, 0, st>>>(s);
  return hipGetLastError();
}

// CV, bias and dV/ds of every walker of a batch into dense arrays (second
// columns hold the contexts' zero second entries for 1-D CVs).
__global__ __launch_bounds__(kBlock) void k_batch_values(const double* const* __restrict__ tab, int32_t W, double* s,
                                                         double* V, double* dV) {
  const int32_t w = blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= W) return;
  const double* sw = tab[3 * w];
  const double* vw = tab[3 * w + 1];
  const double* dw = tab[3 * w + 2];
  if (s) {
    s[2 * w] = sw[0];
    s[2 * w + 1] = sw[1];
  }
  if (V) V[w] = vw[0];
  if (dV) {
    dV[2 * w] = dw[0];
    dV[2 * w + 1] = dw[1];
  }
}

hipError_t launch_batch_values(const double* const* tab, int32_t W, double* s, double* V, double* dV, hipStream_t st) {
  k_batch_values<<<(unsigned)((W + kBlock - 1) / kBlock), kBlock, 0, st>>>(tab, W, s, V, dV);
  return hipGetLastError();
}

hipError_t launch_bias(const BiasArgs& a, int blocks, hipStream_t st) {
  k_bias<<<(unsigned)blocks, blocks > 1 ? kBlock : kBiasBlock, 0, st>>>(a);
  if (blocks > 1) k_bias_finish<<<1, kBlock, 0, st>>>(a, blocks);
  return hipGetLastError();
}

}  // namespace gm
