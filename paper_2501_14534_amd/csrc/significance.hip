// Significance score of Eq. 4, after the ray hits are counted by the
// counting variant of the forward walk (render.hip):
//
//   GS_j = hits_j * o'_j * min(vol_j / v_q, 1)
//
// o'_j = sigmoid(opacity logit) times the hard volume mask (Eq. 3); vol_j =
// the product of the three scales; v_q the volume at ascending rank ceil(q n)
// over all n Gaussians (Sec. 3.2.2 normalises by the volume of the largest
// Gaussians).  Volumes are handled as log-volumes lv = sum of the log-scales
// (monotone, no overflow), so gamma = exp(min(lv - lv_q, 0)).
//
// v_q is found by an exact radix select on the order-preserving 32-bit image
// of lv, 8 bits per pass: each pass histograms the digit of the keys that
// still match the prefix chosen so far (LDS histograms, then one global add
// per non-empty bin), and every workgroup of the next pass (or of the score)
// picks the digit holding the wanted rank for itself from the pass's histogram.
// Four passes, no host round trip, integer counts only: the selected key is
// exact and the result reproducible.  A pass is bound by its global adds, all
// to the same few lines: 256 workgroups of 1024 threads take 8 us for 1M
// Gaussians where 2048 of 256 took 24, and a launch of its own for the pick 5.
#include "gs_common.h"
#include "kernels.h"

namespace gs {

// Order-preserving map of a float to uint32 (negative values reversed); NaN
// goes last.
__device__ __forceinline__ uint32_t order_key(float x) {
  if (x != x) return 0xffffffffu;
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// The same sum in both kernels, so that the selected Gaussian gets gamma = 1.
__device__ __forceinline__ float log_volume(const float* ls, int64_t n, int64_t i) {
  return (ls[i] + ls[n + i]) + ls[2 * n + i];
}

__global__ __launch_bounds__(1024) void select_init_kernel(SelectState* st, uint32_t rank) {
  ((uint32_t*)st->hist)[threadIdx.x] = 0u;
  if (threadIdx.x == 0) {
    st->prefix[0] = 0u;
    st->rank[0] = rank;
  }
}

// The key bits chosen once pass p's histogram is complete, and the rank still
// wanted among the keys that match them: the digit where the running count
// passes the rank.  Called by all threads of a workgroup; its first wave works.
__device__ __forceinline__ uint2 select_pick(const SelectState* st, int p, uint2* s_pick) {
  const int lane = threadIdx.x;
  if (threadIdx.x < kWave) {
    uint32_t c[4], s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      c[k] = st->hist[p][lane * 4 + k];
      s += c[k];
    }
    const uint32_t rank = st->rank[p];
    uint32_t before = wave_inclusive_sum(s) - s;  // keys of lower digits
    int found = -1;
    uint32_t below = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (found < 0 && rank >= before && rank < before + c[k]) {
        found = lane * 4 + k;
        below = before;
      }
      before += c[k];
    }
    if (found >= 0) *s_pick = make_uint2(st->prefix[p] | (uint32_t)found << (24 - 8 * p), rank - below);  // one lane
  }
  __syncthreads();
  return *s_pick;
}

constexpr int kSelectThreads = 1024;
__global__ __launch_bounds__(kSelectThreads) void select_hist_kernel(const float* __restrict__ ls, int64_t n, int p,
                                                                     SelectState* st) {
  __shared__ uint32_t h[256];
  __shared__ uint2 s_pick;
  const int t = threadIdx.x, shift = 24 - 8 * p;
  if (t < 256) h[t] = 0u;
  uint32_t prefix = 0;
  if (p > 0) {
    const uint2 pick = select_pick(st, p - 1, &s_pick);
    prefix = pick.x;
    if (blockIdx.x == 0 && t == 0) {
      st->prefix[p] = pick.x;
      st->rank[p] = pick.y;
    }
  }
  __syncthreads();
  // keys whose bits above this digit equal the prefix chosen so far
  const uint32_t high = p == 0 ? 0u : (0xffffffffu << (shift + 8));
  const int64_t step = (int64_t)gridDim.x * kSelectThreads;
  for (int64_t i = (int64_t)blockIdx.x * kSelectThreads + t; i < n; i += 4 * step) {  // four in flight
    uint32_t k[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) k[q] = i + q * step < n ? order_key(log_volume(ls, n, i + q * step)) : 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (i + q * step < n && ((k[q] ^ prefix) & high) == 0u) atomicAdd(&h[(k[q] >> shift) & 255u], 1u);
  }
  __syncthreads();
  if (t < 256 && h[t] != 0u) atomicAdd(&st->hist[p][t], h[t]);
}

__global__ __launch_bounds__(256) void significance_kernel(const float* __restrict__ ls,
                                                           const float* __restrict__ opacity_logits,
                                                           const float* __restrict__ mask_logits, float mask_thr,
                                                           const uint32_t* __restrict__ hits, int64_t n,
                                                           const SelectState* st, float* __restrict__ score) {
  __shared__ uint2 s_pick;
  const float lvq = key_value(select_pick(st, 3, &s_pick).x);
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t h = hits[i];
  float s = 0.0f;
  if (h != 0u) {
    const float g = __expf(fminf(log_volume(ls, n, i) - lvq, 0.0f));
    float op = sigmoidf(opacity_logits[i]);
    if (mask_logits && !(mask_logits[i] > mask_thr)) op = 0.0f;
    s = (float)h * op * g;
  }
  score[i] = s;
}

hipError_t launch_significance(const float* log_scales, const float* opacity_logits, const float* mask_logits,
                               float mask_thr, const uint32_t* hits, int64_t n, uint32_t rank, SelectState* st,
                               float* score, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(select_init_kernel, dim3(1), dim3(1024), 0, s, st, rank);
  const int64_t want = (n + kSelectThreads - 1) / kSelectThreads;
  const unsigned nb = (unsigned)(want < 256 ? want : 256);
  for (int p = 0; p < 4; ++p)
    hipLaunchKernelGGL(select_hist_kernel, dim3(nb), dim3(kSelectThreads), 0, s, log_scales, n, p, st);
  hipLaunchKernelGGL(significance_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, log_scales,
                     opacity_logits, mask_logits, mask_thr, hits, n, st, score);
  return hipGetLastError();
}

}  // namespace gs
