// Backward of the projection: per-pair splat gradients (u, v, A, B, C, o',
// r, g, b) -> raw Gaussian parameters, accumulated over the V views of the
// call and added (+=) to the caller's gradient arrays.  Straight-through
// estimator for the hard masks (Eq. 3, Eq. 5): d(mask)/d(logit) = sigmoid'.
//
// Three kernels (no atomics):
//   sums:     one wave per 64 consecutive Gaussians and view: each record's pair
//             gradients summed in emission order (double, rounded once to float;
//             the records of a wave own one contiguous run of pairs, whose
//             live rows are staged through LDS); the records with a gradient
//             are packed, with a mask of their lanes (see `slot`);
//   colour:   one thread per Gaussian, the views in order: the SH chain in
//             single precision (diffuse colour, band-mask logits, bands 1..3
//             when that gradient is asked for, and the view-direction term of
//             the mean, left in the record's slot);
//   geometry: one thread per packed record, so that lanes are not idle for the
//             records without a gradient: the EWA chain in double precision (the
//             2x2 inverse amplifies rounding by the condition number of Sigma'):
//     dL/dSigma'  = -Q G_Q Q              (G_Q = [[gA, gB/2], [gB/2, gC]], Q = conic)
//     dL/dSigma   = T^T dL/dSigma' T,     dL/dT = 2 dL/dSigma' T Sigma,  T = J W
//     dL/dJ -> camera-space mean (J's entries, the clamp of the lateral ratios),
//     plus the screen mean (u, v); dL/dmu = W^T dL/dt + colour term;
//     dL/dM = 2 dL/dSigma M with M = Rq diag(s) -> scales, rotation, through
//     the quaternion normalisation; opacity and volume mask.
// Measured at 1M Gaussians in eight views (14.1M pairs, 2.8M walked): 81 + 128 +
// 49 us, 441 us when the colour kernel summed every row of a run and wrote planes
// of all records; at 6M Gaussians in eight views, 16 x 16 tiles, 421 + 670 + 238 us,
// 2.30 ms before.  The colour kernel moves its parameters and gradients at 3.8
// TB/s (a large copy reaches 4.8).
// Each view's contribution is rounded to float and added to the Gaussian's
// totals in view order with non-contracted adds: the association a sequence
// of per-view calls produces, so a batched call equals the per-view calls.
#include "gs_common.h"
#include "kernels.h"

namespace gs {

// Gradient of the 15 SH basis polynomials (k = 1..15) w.r.t. (x, y, z),
// contracted with per-function weights w[k-1]: returns sum_k w_k grad Y_k.
__device__ __forceinline__ void sh_grad15(float x, float y, float z, const float w[15], float* gx, float* gy,
                                          float* gz) {
  const float xx = x * x, yy = y * y, zz = z * z;
  float ax = 0.f, ay = 0.f, az = 0.f;
  // band 1
  ay += -kC1 * w[0];
  az += kC1 * w[1];
  ax += -kC1 * w[2];
  // band 2
  ax += kC2a * y * w[3];
  ay += kC2a * x * w[3];
  ay += -kC2a * z * w[4];
  az += -kC2a * y * w[4];
  ax += -2.f * kC2b * x * w[5];
  ay += -2.f * kC2b * y * w[5];
  az += 4.f * kC2b * z * w[5];
  ax += -kC2a * z * w[6];
  az += -kC2a * x * w[6];
  ax += 2.f * kC2c * x * w[7];
  ay += -2.f * kC2c * y * w[7];
  // band 3
  ax += -6.f * kC3a * x * y * w[8];
  ay += -kC3a * (3.f * xx - 3.f * yy) * w[8];
  ax += kC3b * y * z * w[9];
  ay += kC3b * x * z * w[9];
  az += kC3b * x * y * w[9];
  ax += 2.f * kC3c * x * y * w[10];
  ay += -kC3c * (4.f * zz - xx - 3.f * yy) * w[10];
  az += -8.f * kC3c * y * z * w[10];
  ax += -6.f * kC3d * x * z * w[11];
  ay += -6.f * kC3d * y * z * w[11];
  az += kC3d * (6.f * zz - 3.f * xx - 3.f * yy) * w[11];
  ax += -kC3c * (4.f * zz - 3.f * xx - yy) * w[12];
  ay += 2.f * kC3c * x * y * w[12];
  az += -8.f * kC3c * x * z * w[12];
  ax += 2.f * kC3e * x * z * w[13];
  ay += -2.f * kC3e * y * z * w[13];
  az += kC3e * (xx - yy) * w[13];
  ax += -kC3a * (3.f * xx - 3.f * yy) * w[14];
  ay += 6.f * kC3a * x * y * w[14];
  *gx = ax;
  *gy = ay;
  *gz = az;
}

// t + x without fusing into a preceding multiply (same rounding as two calls).
__device__ __forceinline__ float acc_add(float t, float x) {
#pragma clang fp contract(off)
  return t + x;
}
__device__ __forceinline__ float acc_mul_add(float t, float a, float b) {
#pragma clang fp contract(off)
  const float p = a * b;
  return t + p;
}

// Sums of the 9 pair gradients of each lane's record (cnt pairs from pair
// index off; cnt = 0 gives zeros), accumulated in double and rounded once to
// float.  Called by all 64 lanes of a wave together, for records of
// consecutive Gaussians in one view: their pairs form one contiguous run of
// the [K][9] array (emission order is record order).  A pair the backward walk
// did not reach has no row this step (its live byte is 0) and counts as zero.
//  - Light records (at most kHeavyPairs pairs): window by window of the run, the
//    wave lists the live pairs (their bytes come in one word per lane, a prefix
//    sum over the lanes gives each its place) and loads those rows alone into
//    LDS, three lanes a row.  (Loading its pairs directly would touch a separate
//    cache line per lane and load; four in five pairs of a dense scene are
//    dead, and copying their rows too was half of the reads.)  A record's rows
//    are consecutive there and added in emission order: the first few by the
//    record's own lane, the rest of a longer record by one lane per component
//    (the wave would wait for its longest record's lane otherwise).  Windows
//    holding no light record's pairs are skipped.
//  - Heavy records (the nearest Gaussians cover thousands of tiles, which one
//    lane would add up alone) are left at zero here: the whole wave sums each
//    of them (heavy_sum).
// Both orders depend only on the record's own pairs, not on where its run
// starts, so a record's sums are the same in a batched and a per-view call.
constexpr int kSumWindow = 256;  // pairs per window, four per lane
constexpr int kSumRows = 96;     // rows in LDS at a time: 26 KB a workgroup, six workgroups per CU
constexpr int kSumLong = 14;     // records finished by component at a time: two tasks a lane
constexpr uint32_t kHeavyPairs = 256;
constexpr uint32_t kDirectRows = 6;

template <int ROWS>
struct SumLds {                                  // per wave
  float4 row[ROWS * 3];                          // live rows of the window, three floats in each float4
  uint32_t pre[kWave];                           // per word of live bytes: live pairs before it | its bits << 16
  uint8_t pair[kSumWindow];                      // live row -> pair of the window
  uint32_t rec[kWave];                           // records with more rows than a lane adds alone: those rows,
                                                 // first | end << 16
  double acc[kSumLong][GS_GRAD_FLOATS];          // running sums of kSumLong of them
};

// The pairs [x, y) of the wave's light records (x = y: none).  Offsets grow with
// the lane (consecutive records), so they lie between the first light lane's
// start and the last one's end.
__device__ __forceinline__ uint2 light_run(uint32_t cnt, uint32_t off) {
  const uint32_t lcnt = cnt > kHeavyPairs ? 0u : cnt;
  const uint64_t act = __ballot(lcnt != 0u);
  if (act == 0) return make_uint2(0u, 0u);
  return make_uint2((uint32_t)__builtin_amdgcn_readlane((int)off, __builtin_ctzll(act)),
                    (uint32_t)__builtin_amdgcn_readlane((int)(off + lcnt), 63 - __builtin_clzll(act)));
}

// Live bytes of pairs w0 + 4 lane .. + 3 (w0 a multiple of 4; the array is padded
// past the last pair), for the lanes whose word starts before hi.
__device__ __forceinline__ uint32_t live_word(const uint8_t* __restrict__ live, uint32_t w0, uint32_t hi, int lane) {
  return w0 + 4u * (uint32_t)lane < hi ? *(const uint32_t*)(live + w0 + 4 * lane) : 0u;
}

// `run`: light_run(cnt, off); `word`: live_word of its first window, loaded ahead by the caller.
template <int ROWS>
__device__ __forceinline__ void record_sums(const float* __restrict__ grad_pair, const uint8_t* __restrict__ live,
                                            uint32_t cnt, uint32_t off, uint2 run, uint32_t word, SumLds<ROWS>& s,
                                            int lane, float out[GS_GRAD_FLOATS]) {
  double sum[GS_GRAD_FLOATS] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  const uint32_t lcnt = cnt > kHeavyPairs ? 0u : cnt;
  const uint32_t lo = run.x & ~3u, hi = run.y;  // windows start on whole words of live bytes
  for (uint32_t w0 = lo; w0 < hi; w0 += kSumWindow) {
    const uint32_t w1 = min(w0 + (uint32_t)kSumWindow, hi);
    if (__ballot(lcnt != 0u && off < w1 && off + lcnt > w0) == 0) continue;  // only heavy records' pairs here
    if (w0 != lo) word = live_word(live, w0, hi, lane);
    uint32_t bits = (word & 1u) | ((word >> 7) & 2u) | ((word >> 14) & 4u) | ((word >> 21) & 8u);
    const int left = (int)(w1 - w0) - 4 * lane;  // pairs of this lane's word inside the window
    if (left < 4) bits &= left > 0 ? (1u << left) - 1u : 0u;
    const uint32_t incl = wave_inclusive_sum((uint32_t)__builtin_popcount(bits));
    const uint32_t nl = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    if (nl == 0) continue;  // uniform: no live pair in the window
    uint32_t at = incl - (uint32_t)__builtin_popcount(bits);
    s.pre[lane] = at | (bits << 16);
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if ((bits >> k) & 1u) s.pair[at++] = (uint8_t)(4 * lane + k);
    wave_lds_sync();
    uint32_t r0 = 0, r1 = 0;  // this lane's live rows
    if (lcnt != 0u && off < w1 && off + lcnt > w0) {
      auto rank = [&](uint32_t k) {  // live pairs of the window before pair k
        if (k >= (uint32_t)kSumWindow) return nl;
        const uint32_t q = s.pre[k >> 2];
        return (q & 0xffffu) + (uint32_t)__builtin_popcount((q >> 16) & ((1u << (k & 3u)) - 1u));
      };
      r0 = rank(max(off, w0) - w0);
      r1 = rank(min(off + lcnt, w1) - w0);
    }
    const float* src = grad_pair + (size_t)w0 * GS_GRAD_FLOATS;
    for (uint32_t rb = 0; rb < nl; rb += ROWS) {  // uniform
      // rows straight into LDS, no registers in between: three lanes a row, each
      // 12 bytes into the first three floats of its 16 (the load's lane stride)
      const uint32_t lanes = 3u * min(nl - rb, (uint32_t)ROWS);
      for (uint32_t j = 0; j < lanes; j += kWave) {  // uniform
        const uint32_t e = j + (uint32_t)lane, r = e / 3u;
        if (e < lanes)
          __builtin_amdgcn_global_load_lds(
              (const void*)(src + (uint32_t)s.pair[rb + r] * GS_GRAD_FLOATS + 3u * (e - 3u * r)),
              (__attribute__((address_space(3))) void*)(s.row + j), 12, 0, 0);
      }
      const uint32_t ra = max(r0, rb), re = min(r1, rb + ROWS);
      const uint32_t rd = min(re, ra + kDirectRows);
      const uint64_t more = __ballot(rd < re);
      const uint32_t place = (uint32_t)__popcll(more & ((1ull << lane) - 1ull));
      if (rd < re) s.rec[place] = (rd - rb) | ((re - rb) << 16);
      __builtin_amdgcn_s_waitcnt(0);  // the LDS writes of the loads above have landed
      wave_lds_sync();
      for (uint32_t r = ra; r < rd; ++r)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          const float4 t = s.row[3 * (r - rb) + q];
          sum[3 * q + 0] += (double)t.x;
          sum[3 * q + 1] += (double)t.y;
          sum[3 * q + 2] += (double)t.z;
        }
      const uint32_t nmore = (uint32_t)__popcll(more);
      for (uint32_t p0 = 0; p0 < nmore; p0 += kSumLong) {  // uniform
        const bool mine = rd < re && place - p0 < (uint32_t)kSumLong;
        if (mine)
#pragma unroll
          for (int c = 0; c < GS_GRAD_FLOATS; ++c) s.acc[place - p0][c] = sum[c];
        wave_lds_sync();
        const uint32_t tasks = GS_GRAD_FLOATS * min(nmore - p0, (uint32_t)kSumLong);
        for (uint32_t t = (uint32_t)lane; t < tasks; t += kWave) {
          const uint32_t q = t / GS_GRAD_FLOATS, c = t - q * GS_GRAD_FLOATS, e = s.rec[p0 + q];
          const float* col = (const float*)s.row + c + c / 3u;  // component c of row 0
          double x = s.acc[q][c];
          const uint32_t end = e >> 16;
#pragma unroll 4
          for (uint32_t r = e & 0xffffu; r < end; ++r) x += (double)col[12u * r];
          s.acc[q][c] = x;
        }
        wave_lds_sync();
        if (mine)
#pragma unroll
          for (int c = 0; c < GS_GRAD_FLOATS; ++c) sum[c] = s.acc[place - p0][c];
      }
      wave_lds_sync();  // every lane has read the rows before the next ones overwrite them
    }
  }
#pragma unroll
  for (int c = 0; c < GS_GRAD_FLOATS; ++c) out[c] = (float)sum[c];
}

__device__ __forceinline__ double wave_sum_f64(double x) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) x += __shfl_xor(x, o, kWave);
  return x;
}

// The nine sums of one heavy record (cnt pairs from pair index off), by the
// whole wave: lane j adds pairs j, j + 64, ... in double, a butterfly in a fixed
// pattern adds the lanes, and the sum is rounded once to float.
__device__ __forceinline__ void heavy_sum(const float* __restrict__ grad_pair, const uint8_t* __restrict__ live,
                                          uint32_t cnt, uint32_t off, int lane, float out[GS_GRAD_FLOATS]) {
  double part[GS_GRAD_FLOATS] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
  for (uint32_t j = (uint32_t)lane; j < cnt; j += kWave) {
    const size_t k = (size_t)off + j;
    if (live[k]) {
      const float* row = grad_pair + k * GS_GRAD_FLOATS;
#pragma unroll
      for (int c = 0; c < GS_GRAD_FLOATS; ++c) part[c] += (double)row[c];
    }
  }
#pragma unroll
  for (int c = 0; c < GS_GRAD_FLOATS; ++c) out[c] = (float)wave_sum_f64(part[c]);
}

// What the kernels hand to each other: the nine sums of a record (u, v, A, B, C,
// o', r, g, b), the last three replaced by the colour term of its mean gradient.
// The 64 records of a wave's Gaussians in one view own 64 slots of 12 floats;
// the records with any non-zero sum take them in lane order, in whole 128-byte
// lines, and rec_mask says which lanes they are.  Most records of a dense scene
// have no gradient (one in ten has at 1M Gaussians in eight views): planes of
// all records, zeros included so that lines are written whole, moved 288 MB
// there each way, the slots about a seventh.
constexpr int kSlot = 12;
__device__ __forceinline__ float* slot(const ProjectBwdArgs& b, int v, int64_t wave, int rank) {
  return b.rec + (((size_t)v * (size_t)b.nwaves + (size_t)wave) * kWave + (size_t)rank) * kSlot;
}
__device__ __forceinline__ int rank_of(uint64_t mask, int lane) { return __popcll(mask & ((1ull << lane) - 1ull)); }

// Record sums, one wave per 64 Gaussians and kSumViews views (blockIdx.y).
// Bound by latency: a wave's counts, live bytes and rows are loads that wait for
// each other, a few hundred bytes each, so the counts and the live bytes of its
// views are loaded together where there are waves enough to fill the chip.
template <int kSumViews, int ROWS>
__device__ __forceinline__ void sums_of_wave(const ProjectBwdArgs& b, int V, int v0, int64_t gwave, SumLds<ROWS>& lds) {
  const int64_t n = b.p.n;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t i = gwave * kWave + lane;
  uint32_t cnts[kSumViews], offs[kSumViews], words[kSumViews];
#pragma unroll
  for (int k = 0; k < kSumViews; ++k) {
    const int64_t r = (int64_t)(v0 + k) * n + i;
    const bool use = i < n && v0 + k < V;
    cnts[k] = use ? b.tiles_touched[r] : 0u;
    offs[k] = use ? b.offsets[r] : 0u;
  }
  if (*b.status != 0) {  // overflow: no lists, no gradients
#pragma unroll
    for (int k = 0; k < kSumViews; ++k) cnts[k] = 0u;
  }
  uint2 runs[kSumViews];
#pragma unroll
  for (int k = 0; k < kSumViews; ++k) {
    runs[k] = light_run(cnts[k], offs[k]);
    words[k] = live_word(b.pair_live, runs[k].x & ~3u, runs[k].y, lane);
  }
#pragma unroll
  for (int k = 0; k < kSumViews; ++k) {
    const int v = v0 + k;
    if (v >= V) break;
    const uint32_t cnt = cnts[k], off = offs[k];
    uint64_t mask = 0;
    if (__ballot(cnt != 0u) != 0) {
      float g9[GS_GRAD_FLOATS];
      record_sums(b.grad_pair, b.pair_live, cnt, off, runs[k], words[k], lds, lane, g9);
      for (uint64_t hv = __ballot(cnt > kHeavyPairs); hv; hv &= hv - 1) {
        const int L = __builtin_ctzll(hv);
        float t[GS_GRAD_FLOATS];
        heavy_sum(b.grad_pair, b.pair_live, (uint32_t)__builtin_amdgcn_readlane((int)cnt, L),
                  (uint32_t)__builtin_amdgcn_readlane((int)off, L), lane, t);
#pragma unroll
        for (int c = 0; c < GS_GRAD_FLOATS; ++c) g9[c] = lane == L ? t[c] : g9[c];
      }
      bool some = false;  // a NaN counts
#pragma unroll
      for (int c = 0; c < GS_GRAD_FLOATS; ++c) some |= g9[c] != 0.f;
      if (b.g_mean2d && some) {
        b.g_mean2d[((int64_t)v * 2 + 0) * n + i] += g9[0];
        b.g_mean2d[((int64_t)v * 2 + 1) * n + i] += g9[1];
      }
      mask = __ballot(some);
      float* base = slot(b, v, gwave, 0);
      if (some) {
        float4* o = (float4*)(base + rank_of(mask, lane) * kSlot);
        o[0] = make_float4(g9[0], g9[1], g9[2], g9[3]);
        o[1] = make_float4(g9[4], g9[5], g9[6], g9[7]);
        o[2] = make_float4(g9[8], 0.f, 0.f, 0.f);
      }
      const int used = kSlot * __popcll(mask), pad = -used & 31;  // to the end of the 128-byte line
      if (lane < pad) base[used + lane] = 0.f;
    }
    if (lane == 0) b.rec_mask[(size_t)v * b.nwaves + gwave] = mask;
  }
}

template <int kSumViews>
__global__ __launch_bounds__(256) void project_bwd_sums_kernel(ProjectBwdArgs b, int V) {
  __shared__ SumLds<kSumRows> s_sum[256 / kWave];
  const int wave = threadIdx.x / kWave;
  const int64_t gwave = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave;
  if (gwave < b.nwaves) sums_of_wave<kSumViews>(b, V, (int)blockIdx.y * kSumViews, gwave, s_sum[wave]);
}

// A parameter gradient: written (assign) or added.
__device__ __forceinline__ void grad_out(float* g, bool assign, float t) { *g = assign ? t : *g + t; }

// Colour-kernel outputs of Gaussian i.
template <int DEG, bool REST>
__device__ __forceinline__ void colour_grads_out(const ProjectBwdArgs& b, int64_t n, int64_t i, const float tdc[3],
                                                 const float tbm[3], const float (*trest)[3]) {
  const bool as = b.assign != 0;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (b.g_sh_dc) grad_out(&b.g_sh_dc[k * n + i], as, tdc[k]);
  if (DEG > 0 && b.g_sh_mask_logits && b.p.sh_mask_logits) {
#pragma unroll
    for (int l = 1; l <= DEG; ++l) grad_out(&b.g_sh_mask_logits[(l - 1) * n + i], as, tbm[l - 1]);
  }
  if (REST) {
    constexpr int NR = (DEG + 1) * (DEG + 1) - 1;
#pragma unroll
    for (int k = 1; k <= NR; ++k)
#pragma unroll
      for (int c = 0; c < 3; ++c) grad_out(&b.g_sh_rest[((k - 1) * 3 + c) * n + i], as, trest[k - 1][c]);
  }
}

// Masks of the records with a gradient: word v of a wave's (wave-uniform).
__device__ __forceinline__ uint64_t record_mask(const ProjectBwdArgs& b, int v, int64_t gwave) {
  return b.rec_mask[(size_t)v * (size_t)b.nwaves + (size_t)gwave];
}

// Band masks of Gaussian i (Eq. 5): sigmoid(m_l) > eps <=> m_l > logit(eps).
__device__ __forceinline__ void band_masks(const ProjectArgs& a, int64_t n, int64_t i, float bm[3], bool on[4]) {
  on[0] = on[1] = on[2] = on[3] = true;
  bm[0] = bm[1] = bm[2] = 0.f;
  if (a.sh_mask_logits) {
#pragma unroll
    for (int l = 1; l <= 3; ++l) {
      bm[l - 1] = a.sh_mask_logits[(l - 1) * n + i];
      on[l] = bm[l - 1] > a.sh_mask_thr;
    }
  }
}

// Unit view direction from the camera centre to the mean, and 1 / distance.
__device__ __forceinline__ void view_dir(const ViewArgs& c, const float mu[3], float* dx, float* dy, float* dz,
                                        float* il) {
  const float d0 = mu[0] - c.campos[0], d1 = mu[1] - c.campos[1], d2 = mu[2] - c.campos[2];
  *il = 1.0f / sqrtf(d0 * d0 + d1 * d1 + d2 * d2);
  *dx = d0 * *il, *dy = d1 * *il, *dz = d2 * *il;
}

// Per Gaussian over the views with a gradient: the colour chain: the gradient
// of the clamped colour, the diffuse colour and band-mask gradients, with REST
// the SH bands 1..DEG (sum over the views of Y_k(d_v) times that gradient; bands
// whose hard mask is off get nothing), and the colour term of the mean gradient
// (through the view direction).
template <int DEG, bool REST>
__device__ __forceinline__ void colour_of_wave(const ProjectBwdArgs& b, const ViewTable& vt) {
  const ProjectArgs& a = b.p;
  const int64_t n = a.n;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = threadIdx.x & (kWave - 1);
  // the wave of Gaussians, in a scalar register: masks are scalar loads
  const int64_t gwave = (int64_t)blockIdx.x * (blockDim.x / kWave) +
                        __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  if (gwave >= b.nwaves) return;
  const bool valid = i < n;
  const int V = vt.nviews;
  constexpr int NRT = REST ? (DEG + 1) * (DEG + 1) - 1 : 1;
  const float zero3[3] = {0.f, 0.f, 0.f};
  float trest[NRT][3];
#pragma unroll
  for (int k = 0; k < NRT; ++k) trest[k][0] = trest[k][1] = trest[k][2] = 0.f;
  // no gradient in the whole wave (culled, off-screen, not reached, or the
  // binning overflowed): zeros when the gradients are written, else nothing
  uint64_t any = 0;
  for (int v = 0; v < V; ++v) any |= record_mask(b, v, gwave);
  if (any == 0) {
    if (b.assign && valid) colour_grads_out<DEG, REST>(b, n, i, zero3, zero3, trest);
    return;
  }
  const bool vis = (any >> lane) & 1ull;

  constexpr int NR = DEG > 0 ? (DEG + 1) * (DEG + 1) - 1 : 1;
  float mu[3] = {0.f, 0.f, 0.f}, dc[3] = {0.f, 0.f, 0.f};
  float rest[NR][3];
  float bm[3] = {0.f, 0.f, 0.f};
  bool band_on[4] = {true, true, true, true};
#pragma unroll
  for (int k = 0; k < NR; ++k) rest[k][0] = rest[k][1] = rest[k][2] = 0.f;
  if (vis) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      mu[k] = a.means[k * n + i];
      dc[k] = a.sh_dc[k * n + i];
    }
    band_masks(a, n, i, bm, band_on);
    if (DEG > 0) {
      // every band's coefficients are read: the band-mask gradient needs them
      // even when the band is off (straight-through estimator)
#pragma unroll
      for (int k = 1; k <= NR; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) rest[k - 1][c] = a.sh_rest[((k - 1) * 3 + c) * n + i];
    }
  }
  float tdc[3] = {0.f, 0.f, 0.f}, tbm[3] = {0.f, 0.f, 0.f};

  // v is the same in every lane: camera constants are scalar loads
  for (int v = 0; v < V; ++v) {
    const uint64_t mask = record_mask(b, v, gwave);
    if (mask == 0) continue;
    if (!((mask >> lane) & 1ull)) continue;
    float* rec = slot(b, v, gwave, rank_of(mask, lane));
    float gmu_col[3] = {0.f, 0.f, 0.f};
    const float grgb[3] = {rec[6], rec[7], rec[8]};
    if (grgb[0] != 0.f || grgb[1] != 0.f || grgb[2] != 0.f) {
      const ViewArgs& c = vt.v[v];
      float pre[3] = {dc[0], dc[1], dc[2]};
      float Y[15];
      float dx = 0.f, dy = 0.f, dz = 0.f, il = 1.f;
      if (DEG > 0) {
        view_dir(c, mu, &dx, &dy, &dz, &il);
        sh_basis15(dx, dy, dz, Y);
        // flat loops with constant trip counts keep rest/Y in registers
#pragma unroll
        for (int k = 1; k < kShCoeffs; ++k) {
          const int l = sh_band(k);
          if (l > DEG || !band_on[l]) continue;
#pragma unroll
          for (int ch = 0; ch < 3; ++ch) pre[ch] += Y[k - 1] * rest[k - 1][ch];
        }
      }
      float gpre[3];
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        gpre[ch] = pre[ch] < 0.f ? 0.f : grgb[ch];
        tdc[ch] = acc_add(tdc[ch], gpre[ch]);
      }
      if (DEG > 0) {
        float wY[15];
#pragma unroll
        for (int k = 0; k < 15; ++k) wY[k] = 0.f;
        float band[3] = {0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 1; k < kShCoeffs; ++k) {
          const int l = sh_band(k);
          if (l > DEG) continue;
          const float cg = rest[k - 1][0] * gpre[0] + rest[k - 1][1] * gpre[1] + rest[k - 1][2] * gpre[2];
          band[l - 1] += Y[k - 1] * cg;
          if (band_on[l]) wY[k - 1] = cg;
        }
#pragma unroll
        for (int l = 1; l <= DEG; ++l) {
          const float sb = sigmoidf(bm[l - 1]);
          tbm[l - 1] = acc_mul_add(tbm[l - 1], band[l - 1], sb * (1.f - sb));
        }
        float gdx, gdy, gdz;
        sh_grad15(dx, dy, dz, wY, &gdx, &gdy, &gdz);
        const float dot = dx * gdx + dy * gdy + dz * gdz;
        gmu_col[0] = (gdx - dx * dot) * il;
        gmu_col[1] = (gdy - dy * dot) * il;
        gmu_col[2] = (gdz - dz * dot) * il;
        if (REST && (gpre[0] != 0.f || gpre[1] != 0.f || gpre[2] != 0.f)) {  // else it adds exact zeros
#pragma unroll
          for (int k = 1; k < kShCoeffs; ++k) {
            const int l = sh_band(k);
            if (l > DEG || !band_on[l]) continue;
#pragma unroll
            for (int ch = 0; ch < 3; ++ch)
              trest[k - 1][ch] = acc_mul_add(trest[k - 1][ch], Y[k - 1], gpre[ch]);
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) rec[6 + k] = gmu_col[k];
  }

  if (!valid || (!vis && !b.assign)) return;
  colour_grads_out<DEG, REST>(b, n, i, tdc, tbm, trest);
}

template <int DEG, bool REST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void project_bwd_color_kernel(
    ProjectBwdArgs b, ViewTable vt) {
  colour_of_wave<DEG, REST>(b, vt);
}

// Geometry-kernel outputs of Gaussian i.
__device__ __forceinline__ void geom_grads_out(const ProjectBwdArgs& b, int64_t n, int64_t i, const float* tmu,
                                               const float* tls, const float* tq, float top, float tmask) {
  const bool as = b.assign != 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    if (b.g_means) grad_out(&b.g_means[k * n + i], as, tmu[k]);
    if (b.g_log_scales) grad_out(&b.g_log_scales[k * n + i], as, tls[k]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (b.g_quats) grad_out(&b.g_quats[k * n + i], as, tq[k]);
  if (b.g_opacity_logits) grad_out(&b.g_opacity_logits[i], as, top);
  if (b.g_mask_logits && b.p.mask_logits) grad_out(&b.g_mask_logits[i], as, tmask);
}

// Lane of the k-th set bit of m (k < popcount).
__device__ __forceinline__ int select_lane(uint64_t m, int k) {
  uint32_t x = (uint32_t)m;
  int base = 0;
  const int c0 = __popc(x);
  if (k >= c0) k -= c0, x = (uint32_t)(m >> 32), base = 32;
#pragma unroll
  for (int s = 16; s > 0; s >>= 1) {
    const int c = __popc(x & ((1u << s) - 1u));
    if (k >= c) k -= c, x >>= s, base += s;
  }
  return base;
}

constexpr int kGeomOut = 12;  // mean 3, log-scale 3, quaternion 4, opacity logit, mask logit

// The geometry chain of record (v, i): its contributions to the gradients of
// Gaussian i, each rounded to float.
__device__ __forceinline__ void geom_record(const ProjectArgs& a, const ViewArgs& c, int64_t i,
                                            const float* __restrict__ rp, float out[kGeomOut]) {
  const int64_t n = a.n;
  const double gu = rp[0], gv = rp[1], gA = rp[2], gB = rp[3], gC = rp[4], go = rp[5];
  const float cmu[3] = {rp[6], rp[7], rp[8]};  // colour term of the mean gradient
#pragma unroll
  for (int k = 0; k < kGeomOut; ++k) out[k] = 0.f;
  if (gu == 0.0 && gv == 0.0 && gA == 0.0 && gB == 0.0 && gC == 0.0 && go == 0.0 && cmu[0] == 0.f && cmu[1] == 0.f &&
      cmu[2] == 0.f)
    return;
  float mu[3], ls[3], q[4];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    mu[k] = a.means[k * n + i];
    ls[k] = a.log_scales[k * n + i];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) q[k] = a.quats[k * n + i];
  const float ol = a.opacity_logits[i];

  const double q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
  const double iq = 1.0 / sqrt(q0 * q0 + q1 * q1 + q2 * q2 + q3 * q3);
  const double w = q0 * iq, x = q1 * iq, y = q2 * iq, z = q3 * iq;
  const double Rq[3][3] = {{1.0 - 2.0 * (y * y + z * z), 2.0 * (x * y - w * z), 2.0 * (x * z + w * y)},
                           {2.0 * (x * y + w * z), 1.0 - 2.0 * (x * x + z * z), 2.0 * (y * z - w * x)},
                           {2.0 * (x * z - w * y), 2.0 * (y * z + w * x), 1.0 - 2.0 * (x * x + y * y)}};
  double s[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) s[k] = exp((double)ls[k]);
  double Sig[6];  // xx, xy, xz, yy, yz, zz
  {
    double M[3][3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
      for (int k = 0; k < 3; ++k) M[r][k] = Rq[r][k] * s[k];
    Sig[0] = M[0][0] * M[0][0] + M[0][1] * M[0][1] + M[0][2] * M[0][2];
    Sig[1] = M[0][0] * M[1][0] + M[0][1] * M[1][1] + M[0][2] * M[1][2];
    Sig[2] = M[0][0] * M[2][0] + M[0][1] * M[2][1] + M[0][2] * M[2][2];
    Sig[3] = M[1][0] * M[1][0] + M[1][1] * M[1][1] + M[1][2] * M[1][2];
    Sig[4] = M[1][0] * M[2][0] + M[1][1] * M[2][1] + M[1][2] * M[2][2];
    Sig[5] = M[2][0] * M[2][0] + M[2][1] * M[2][1] + M[2][2] * M[2][2];
  }
  const double op = 1.0 / (1.0 + exp(-(double)ol));
  double sm = 0.0;
  if (a.mask_logits) sm = 1.0 / (1.0 + exp(-(double)a.mask_logits[i]));

    const double fx = c.fx, fy = c.fy;
    const double t0 = (double)c.R[0] * mu[0] + (double)c.R[1] * mu[1] + (double)c.R[2] * mu[2] + (double)c.t[0];
    const double t1 = (double)c.R[3] * mu[0] + (double)c.R[4] * mu[1] + (double)c.R[5] * mu[2] + (double)c.t[1];
    const double t2 = (double)c.R[6] * mu[0] + (double)c.R[7] * mu[1] + (double)c.R[8] * mu[2] + (double)c.t[2];
    const double iz = 1.0 / t2;
    const double ux = t0 * iz, uy = t1 * iz;
    const double lx = c.limx, ly = c.limy;
    const bool inx = ux >= -lx && ux <= lx;
    const bool iny = uy >= -ly && uy <= ly;
    const double rx = fmin(fmax(ux, -lx), lx);
    const double ry = fmin(fmax(uy, -ly), ly);
    const double j00 = fx * iz, j02 = -fx * rx * iz, j11 = fy * iz, j12 = -fy * ry * iz;
    double Tm[2][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      Tm[0][k] = j00 * (double)c.R[k] + j02 * (double)c.R[6 + k];
      Tm[1][k] = j11 * (double)c.R[3 + k] + j12 * (double)c.R[6 + k];
    }
    double TS[2][3];  // T Sigma
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
      TS[rr][0] = Tm[rr][0] * Sig[0] + Tm[rr][1] * Sig[1] + Tm[rr][2] * Sig[2];
      TS[rr][1] = Tm[rr][0] * Sig[1] + Tm[rr][1] * Sig[3] + Tm[rr][2] * Sig[4];
      TS[rr][2] = Tm[rr][0] * Sig[2] + Tm[rr][1] * Sig[4] + Tm[rr][2] * Sig[5];
    }
    const double ca = TS[0][0] * Tm[0][0] + TS[0][1] * Tm[0][1] + TS[0][2] * Tm[0][2] + (double)c.lowpass;
    const double cb = TS[0][0] * Tm[1][0] + TS[0][1] * Tm[1][1] + TS[0][2] * Tm[1][2];
    const double cc = TS[1][0] * Tm[1][0] + TS[1][1] * Tm[1][1] + TS[1][2] * Tm[1][2] + (double)c.lowpass;
    const double idet = 1.0 / (ca * cc - cb * cb);
    const double QA = cc * idet, QB = -cb * idet, QC = ca * idet;
    // dL/dSigma' = -Q G_Q Q
    const double P00 = QA * gA + QB * 0.5 * gB, P01 = QA * 0.5 * gB + QB * gC;
    const double P10 = QB * gA + QC * 0.5 * gB, P11 = QB * 0.5 * gB + QC * gC;
    const double G00 = -(P00 * QA + P01 * QB);
    const double G01 = -(P00 * QB + P01 * QC);
    const double G11 = -(P10 * QB + P11 * QC);
    // dL/dT = 2 G T Sigma; T = J W with J00, J02, J11, J12 varying
    double gT[2][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      gT[0][k] = 2.0 * (G00 * TS[0][k] + G01 * TS[1][k]);
      gT[1][k] = 2.0 * (G01 * TS[0][k] + G11 * TS[1][k]);
    }
    const double gj00 = gT[0][0] * c.R[0] + gT[0][1] * c.R[1] + gT[0][2] * c.R[2];
    const double gj02 = gT[0][0] * c.R[6] + gT[0][1] * c.R[7] + gT[0][2] * c.R[8];
    const double gj11 = gT[1][0] * c.R[3] + gT[1][1] * c.R[4] + gT[1][2] * c.R[5];
    const double gj12 = gT[1][0] * c.R[6] + gT[1][1] * c.R[7] + gT[1][2] * c.R[8];
    const double iz2 = iz * iz;
    double gt0 = gu * fx * iz, gt1 = gv * fy * iz;
    double gt2 = -gu * fx * t0 * iz2 - gv * fy * t1 * iz2;
    gt2 += -gj00 * fx * iz2 - gj11 * fy * iz2;
    // J02 = -fx rx / z, rx = clamp(x / z): d/dx = -fx/z^2 (unclamped); d/dz = fx rx/z^2 (+ fx x/z^3 unclamped)
    gt2 += gj02 * fx * rx * iz2 + gj12 * fy * ry * iz2;
    if (inx) {
      gt0 += -gj02 * fx * iz2;
      gt2 += gj02 * fx * t0 * iz2 * iz;
    }
    if (iny) {
      gt1 += -gj12 * fy * iz2;
      gt2 += gj12 * fy * t1 * iz2 * iz;
    }
    // dL/dSigma = T^T G T (symmetric), then dL/dM = (G + G^T) M = 2 G M
    double gS[3][3];
#pragma unroll
    for (int rr = 0; rr < 3; ++rr)
#pragma unroll
      for (int k = 0; k < 3; ++k)
        gS[rr][k] = Tm[0][rr] * (G00 * Tm[0][k] + G01 * Tm[1][k]) + Tm[1][rr] * (G01 * Tm[0][k] + G11 * Tm[1][k]);
    double gsc[3], gR[3][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double acc[3];
#pragma unroll
      for (int rr = 0; rr < 3; ++rr)
        acc[rr] = (gS[rr][0] + gS[0][rr]) * Rq[0][k] * s[k] + (gS[rr][1] + gS[1][rr]) * Rq[1][k] * s[k] +
                  (gS[rr][2] + gS[2][rr]) * Rq[2][k] * s[k];
      gsc[k] = acc[0] * Rq[0][k] + acc[1] * Rq[1][k] + acc[2] * Rq[2][k];
      gR[0][k] = acc[0] * s[k];
      gR[1][k] = acc[1] * s[k];
      gR[2][k] = acc[2] * s[k];
    }
    const double gw = 2.0 * (-z * gR[0][1] + y * gR[0][2] + z * gR[1][0] - x * gR[1][2] - y * gR[2][0] + x * gR[2][1]);
    const double gx = 2.0 * (y * gR[0][1] + z * gR[0][2] + y * gR[1][0] - 2.0 * x * gR[1][1] - w * gR[1][2] +
                             z * gR[2][0] + w * gR[2][1] - 2.0 * x * gR[2][2]);
    const double gy = 2.0 * (-2.0 * y * gR[0][0] + x * gR[0][1] + w * gR[0][2] + x * gR[1][0] + z * gR[1][2] -
                             w * gR[2][0] + z * gR[2][1] - 2.0 * y * gR[2][2]);
    const double gz = 2.0 * (-2.0 * z * gR[0][0] - w * gR[0][1] + x * gR[0][2] + w * gR[1][0] - 2.0 * z * gR[1][1] +
                             y * gR[1][2] + x * gR[2][0] + y * gR[2][1]);
    const double qd = w * gw + x * gx + y * gy + z * gz;
    // rounded to float; the caller adds the views in order
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double gmu = (double)c.R[k] * gt0 + (double)c.R[3 + k] * gt1 + (double)c.R[6 + k] * gt2;
      out[k] = (float)(gmu + (double)cmu[k]);
      out[3 + k] = (float)(gsc[k] * s[k]);
    }
    out[6] = (float)((gw - w * qd) * iq);
    out[7] = (float)((gx - x * qd) * iq);
    out[8] = (float)((gy - y * qd) * iq);
    out[9] = (float)((gz - z * qd) * iq);
    out[10] = (float)(go * op * (1.0 - op));
    if (a.mask_logits)  // o' = M o, s' = M s (M = 1 here): dL/dM = o dL/do' + sum_k s_k dL/ds'_k
      out[11] = (float)((go * op + gsc[0] * s[0] + gsc[1] * s[1] + gsc[2] * s[2]) * sm * (1.0 - sm));
}

// Geometry: a workgroup owns 256 Gaussians and takes their packed records, view
// by view, 256 at a time, one per thread; the results wait in LDS until each
// thread has added its own Gaussian's, in view order.  Bound by the double
// precision chain (some 600 operations a record): one thread per Gaussian, views
// in turn, ran it with the one lane in ten that had a gradient.
__device__ __forceinline__ void geometry_of_block(const ProjectBwdArgs& b, const ViewTable& vt) {
  constexpr int kWaves = 256 / kWave;
  __shared__ ViewArgs s_view[GS_MAX_VIEWS];
  __shared__ uint64_t s_mask[GS_MAX_VIEWS * kWaves];      // [view][wave]
  __shared__ uint32_t s_pre[GS_MAX_VIEWS * kWaves + 1];   // records before them; the total last
  __shared__ float s_out[256][kGeomOut + 1];
  static_assert(GS_MAX_VIEWS * kWaves <= kWave, "one wave scans the masks");
  const ProjectArgs& a = b.p;
  const int64_t n = a.n;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave, V = vt.nviews;
  const int64_t w0 = (int64_t)blockIdx.x * kWaves, i = (int64_t)blockIdx.x * 256 + t;
  if (wave == 0) {
    const int64_t gw = w0 + lane % kWaves;
    const uint64_t m = lane < V * kWaves && gw < b.nwaves ? record_mask(b, lane / kWaves, gw) : 0ull;
    const uint32_t c = (uint32_t)__popcll(m), incl = wave_inclusive_sum(c);
    s_mask[lane] = m;
    s_pre[lane] = incl - c;
    if (lane == kWave - 1) s_pre[kWave] = incl;
  } else {
    constexpr int kWords = sizeof(ViewArgs) / 4;
    for (int q = t - kWave; q < V * kWords; q += 256 - kWave) ((uint32_t*)s_view)[q] = ((const uint32_t*)vt.v)[q];
  }
  __syncthreads();
  const uint32_t total = s_pre[kWave];
  float sum[kGeomOut];
#pragma unroll
  for (int k = 0; k < kGeomOut; ++k) sum[k] = 0.f;
  bool some = false;
  for (uint32_t base = 0; base < total; base += 256) {  // uniform
    const uint32_t r = base + (uint32_t)t;
    if (r < total) {
      int q = 0;  // the last (view, wave) whose first record is at or before r
#pragma unroll
      for (int s = kWave / 2; s > 0; s >>= 1)
        if (s_pre[q + s] <= r) q += s;
      const int rk = (int)(r - s_pre[q]), v = q / kWaves;
      const int64_t gw = w0 + q % kWaves;
      float out[kGeomOut];
      geom_record(a, s_view[v], gw * kWave + select_lane(s_mask[q], rk), slot(b, v, gw, rk), out);
#pragma unroll
      for (int k = 0; k < kGeomOut; ++k) s_out[t][k] = out[k];
    }
    __syncthreads();
    for (int v = 0; v < V; ++v) {
      const uint64_t m = s_mask[v * kWaves + wave];
      if (!((m >> lane) & 1ull)) continue;
      const uint32_t at = s_pre[v * kWaves + wave] + (uint32_t)rank_of(m, lane) - base;
      if (at >= 256u) continue;  // another chunk's
      some = true;
#pragma unroll
      for (int k = 0; k < kGeomOut; ++k) sum[k] = acc_add(sum[k], s_out[at][k]);
    }
    __syncthreads();
  }
  if (i >= n || (!some && !b.assign)) return;
  geom_grads_out(b, n, i, sum, sum + 3, sum + 6, sum[10], sum[11]);
}

__global__ __launch_bounds__(256, 3) void project_bwd_geom_kernel(ProjectBwdArgs b, ViewTable vt) {
  geometry_of_block(b, vt);
}

// The three stages in one launch: each works on the slots of the workgroup's
// own 256 Gaussians.  For one view and no more workgroups than CUs, where a
// launch costs as much as a stage (2K Gaussians: three kernels of 17 us in
// all); more views would run one after the other, and more Gaussians want the
// occupancy that each stage has on its own.
template <int DEG, bool REST>
__global__ __launch_bounds__(256) void project_bwd_small_kernel(ProjectBwdArgs b, ViewTable vt) {
  __shared__ SumLds<kSumWindow> s_sum[256 / kWave];  // a whole window at once
  const int wave = threadIdx.x / kWave;
  const int64_t gwave = (int64_t)blockIdx.x * (blockDim.x / kWave) + wave;
  if (gwave < b.nwaves) sums_of_wave<1>(b, 1, 0, gwave, s_sum[wave]);
  __syncthreads();
  colour_of_wave<DEG, REST>(b, vt);
  __syncthreads();
  geometry_of_block(b, vt);
}

template <int DEG, bool REST>
static void launch_stages(const ProjectBwdArgs& a, const ViewTable& vt, hipStream_t s) {
  const dim3 block(256), grid((unsigned)((a.p.n + 255) / 256));
  if (vt.nviews == 1 && grid.x <= 256) {
    hipLaunchKernelGGL((project_bwd_small_kernel<DEG, REST>), grid, block, 0, s, a, vt);
    return;
  }
  // one view a wave until that gives more than the 4096 waves that run at once
  if (a.nwaves * vt.nviews > 4 * 4096)
    hipLaunchKernelGGL(project_bwd_sums_kernel<4>, dim3(grid.x, (unsigned)((vt.nviews + 3) / 4)), block, 0, s, a,
                       (int)vt.nviews);
  else
    hipLaunchKernelGGL(project_bwd_sums_kernel<1>, dim3(grid.x, (unsigned)vt.nviews), block, 0, s, a, (int)vt.nviews);
  hipLaunchKernelGGL((project_bwd_color_kernel<DEG, REST>), grid, block, 0, s, a, vt);
  hipLaunchKernelGGL(project_bwd_geom_kernel, grid, block, 0, s, a, vt);
}

hipError_t launch_project_bwd(const ProjectBwdArgs& a, const ViewTable& vt, int deg, hipStream_t s) {
  if (a.p.n == 0) return hipSuccess;
  const bool rest = a.g_sh_rest != nullptr && deg > 0;
  switch (deg) {
    case 0: launch_stages<0, false>(a, vt, s); break;
    case 1: rest ? launch_stages<1, true>(a, vt, s) : launch_stages<1, false>(a, vt, s); break;
    case 2: rest ? launch_stages<2, true>(a, vt, s) : launch_stages<2, false>(a, vt, s); break;
    default: rest ? launch_stages<3, true>(a, vt, s) : launch_stages<3, false>(a, vt, s); break;
  }
  return hipGetLastError();
}

}  // namespace gs
