// Photometric loss of Eq. 7 (the L1 and D-SSIM terms) and its gradient with
// respect to the rendered image, over all views of a call.
//
//   L_v = (1 - lambda) mean|x - y| + lambda (1 - mean S),   L = mean_v L_v
//
// S is the SSIM map of each colour plane from Gaussian-weighted local moments
// (11 x 11 window = outer product of two 11-tap Gaussians of standard deviation
// 1.5, as Sec. 3.2.5 describes; zero padding; C1 = 0.01^2, C2 = 0.03^2).
//
// Two passes over 116 x 16 output tiles, one workgroup of 256 threads per
// (view, plane, tile); both filter columns first, straight from memory into
// registers (a thread owns one of 128 columns, 5 of halo on either side, and 8
// rows; its 18 loads are all in flight together), leave the column sums in LDS,
// and filter rows from there, 4 neighbouring pixels a thread from 16-byte reads:
//   ssim_fwd: the five moments mu_x, mu_y, E[xx], E[yy], E[xy]; S and its
//             partial derivatives dS/dmu_x, dS/dE[xx], dS/dE[xy] (written to
//             the workspace as three planes); per-workgroup sums of S and
//             |x - y|;
//   ssim_bwd: the window's correlation of the three partial-derivative maps
//             (the window is symmetric, so this is the adjoint of the forward
//             filtering), combined per pixel as
//             dS/dx = w*A + 2 x (w*B) + y (w*C), then the L1 term.
// Vector arithmetic bounds both (about 170 and 90 operations a pixel).  Staging
// tiles of 32 x 32 with their halo and reading every tap from LDS was bound by
// those reads (90 and 60 a pixel, now 25 and 15), and the maps as triples were
// written at a stride of 12 bytes.
// One workgroup per view adds its workgroups' sums in a fixed order (double)
// into the view's loss; a last kernel takes their mean.  No atomics:
// reproducible.  (One workgroup for both, a wave per view, took 8-10 us against
// 9 for the two.)
// Measured over eight views of 3.09 Mpix together: forward 141 -> 70 us,
// backward 81 -> 41 us.
#include "gs_common.h"
#include "kernels.h"

namespace gs {

constexpr int kLW = kLossTileW, kLH = kLossTileH;  // output tile: 116 x 16
constexpr int kLR = 5;                  // window radius
constexpr int kTaps = 2 * kLR + 1;
constexpr int kCols = 128;              // columns filtered: kLW + 2 kLR, rounded up to two waves
constexpr int kRows = kLH / 2;          // output rows of a thread's column (two halves of the workgroup)
constexpr int kQ = 4;                   // neighbouring output pixels per thread of the row pass
constexpr float kSsimC1 = 0.0001f;      // (0.01)^2
constexpr float kSsimC2 = 0.0009f;      // (0.03)^2
// the last group's 16-byte reads end inside the row: 4 (kLW / 4 - 1) + 16 <= kCols
static_assert(kLW % kQ == 0 && kLW / kQ <= 32 && kLW - kQ + 16 <= kCols && kLW + 2 * kLR <= kCols, "tile width");

typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any float's address

// Workgroup b's tile: consecutive workgroups go to the 8 XCDs in turn, so each
// XCD takes a run of neighbouring tiles, whose halos meet in its L2.
__device__ __forceinline__ int xcd_run(int b, int nb) {
  const int per = nb / 8, rest = nb - 8 * per, x = b & 7;
  return b / 8 + x * per + min(x, rest);
}

// Thread t's column (t % 128 of the tile's window) and first staged row, and
// which of its rows are inside the image (the rows of a wave are the same).
struct Column {
  int x, y;
  bool in;
};
__device__ __forceinline__ Column column_of(int t, int x0, int y0, int W) {
  Column c;
  c.x = (int)((uint32_t)x0 - kLR + (t & (kCols - 1)));  // past the largest int: negative
  c.y = y0 - kLR + __builtin_amdgcn_readfirstlane(t / kCols) * kRows;
  c.in = (uint32_t)c.x < (uint32_t)W;
  return c;
}

// The column's kRows + 10 values of a plane, zero outside the image.
__device__ __forceinline__ void load_column(const float* __restrict__ plane, const Column& c, int W, int H,
                                            float v[kRows + 2 * kLR]) {
#pragma unroll
  for (int i = 0; i < kRows + 2 * kLR; ++i) {
    const uint32_t y = (uint32_t)c.y + (uint32_t)i;  // rows above the image wrap to the end
    v[i] = 0.0f;
    if (y < (uint32_t)H && c.in) v[i] = (plane + (int64_t)y * W)[c.x];
  }
}

// Row sums of the four pixels at columns 4 g .. 4 g + 3 from a row of column sums.
__device__ __forceinline__ void filter_row(const float* row, int g, const float* taps, float out[kQ]) {
  float v[16];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float4 f = ((const float4*)row)[g + k];
    v[4 * k] = f.x, v[4 * k + 1] = f.y, v[4 * k + 2] = f.z, v[4 * k + 3] = f.w;
  }
#pragma unroll
  for (int p = 0; p < kQ; ++p) {
    out[p] = 0.0f;
#pragma unroll
    for (int k = 0; k < kTaps; ++k) out[p] += taps[k] * v[p + k];
  }
}

// Up to four neighbouring floats (m of them inside the image's row).
__device__ __forceinline__ Quad load_quad(const float* p, int m) {
  if (m >= kQ) return *(const Quad*)p;
  Quad q = {0.f, 0.f, 0.f, 0.f};
  q.x = p[0];
  if (m > 1) q.y = p[1];
  if (m > 2) q.z = p[2];
  return q;
}
__device__ __forceinline__ void store_quad(float* p, int m, Quad q) {
  if (m >= kQ) {
    *(Quad*)p = q;
    return;
  }
  p[0] = q.x;
  if (m > 1) p[1] = q.y;
  if (m > 2) p[2] = q.z;
}

// 40 KB of LDS: four workgroups share a CU.
__global__ __launch_bounds__(256, 4) void ssim_fwd_kernel(const float* __restrict__ image,
                                                          const float* __restrict__ target, LossViews lv,
                                                          float* __restrict__ dmap, int64_t map_stride,
                                                          float* __restrict__ bsum, int first) {
  __shared__ float4 s_v4[5 * kLH * kCols / 4];
  float* s_v = (float*)s_v4;
  const int b = xcd_run(first + (int)blockIdx.x, lv.total_blocks);
  const LossTile tl = loss_tile(lv, b);
  const LossView& q = lv.v[tl.view];
  const int W = q.W, H = q.H, t = threadIdx.x;
  const int64_t plane_px = (int64_t)W * H;
  const int64_t poff = 3 * q.pix_off + tl.plane * plane_px;  // this plane in the view-concatenated layout
  const float* xp = image + poff;
  const float* yp = target + poff;
  const int x0 = tl.tx * q.tw, y0 = tl.ty * kLH;
  {  // column pass
    const Column c = column_of(t, x0, y0, W);
    float x[kRows + 2 * kLR], y[kRows + 2 * kLR];
    load_column(xp, c, W, H, x);
    load_column(yp, c, W, H, y);
    float acc[5][kRows];
#pragma unroll
    for (int i = 0; i < kRows + 2 * kLR; ++i) {
      const float m[5] = {x[i], y[i], x[i] * x[i], y[i] * y[i], x[i] * y[i]};
#pragma unroll
      for (int r = 0; r < kRows; ++r) {  // row r's taps are the staged rows r .. r + 10
        if (i < r || i > r + 2 * kLR) continue;
#pragma unroll
        for (int e = 0; e < 5; ++e) acc[e][r] = i == r ? lv.g[0] * m[e] : acc[e][r] + lv.g[i - r] * m[e];
      }
    }
    const int row0 = (t / kCols) * kRows, col = t & (kCols - 1);
#pragma unroll
    for (int e = 0; e < 5; ++e)
#pragma unroll
      for (int r = 0; r < kRows; ++r) s_v[(e * kLH + row0 + r) * kCols + col] = acc[e][r];
  }
  __syncthreads();
  // row pass: 8 rows of 32 threads (29 with pixels), twice
  const int g = t & 31, px = x0 + kQ * g;
  const int m = kQ * g < q.tw ? (W - x0) - kQ * g : 0;  // (x0 + 4 g may pass the largest int: compare from below)
  float s_val = 0.f, l1 = 0.f;
#pragma unroll 1
  for (int oy = t / 32; oy < kLH; oy += 8) {
    const int py = y0 + oy;
    if (m <= 0 || py >= H) continue;
    float f[5][kQ];
#pragma unroll
    for (int e = 0; e < 5; ++e) filter_row(s_v + (e * kLH + oy) * kCols, g, lv.g, f[e]);
    const int64_t pix = poff + (int64_t)py * W + px;
    const Quad x = load_quad(image + pix, m), y = load_quad(target + pix, m);
    Quad da, db, dc;
#pragma unroll
    for (int p = 0; p < kQ; ++p) {
      const float mx = f[0][p], my = f[1][p];
      const float sxx = f[2][p] - mx * mx, syy = f[3][p] - my * my, sxy = f[4][p] - mx * my;
      const float n1 = 2.f * mx * my + kSsimC1, n2 = 2.f * sxy + kSsimC2;
      const float d1 = mx * mx + my * my + kSsimC1, d2 = sxx + syy + kSsimC2;
      const float id = 1.0f / (d1 * d2);
      const float S = n1 * n2 * id;
      da[p] = 2.f * my * (n2 - n1) * id - 2.f * mx * S * ((d2 - d1) * id);  // 1/d1 - 1/d2
      db[p] = -S * (d1 * id);
      dc[p] = 2.f * n1 * id;
      if (p < m) {
        s_val += S;
        l1 += fabsf(x[p] - y[p]);
      }
    }
    store_quad(dmap + pix, m, da);
    store_quad(dmap + map_stride + pix, m, db);
    store_quad(dmap + 2 * map_stride + pix, m, dc);
  }
  // fixed-order block sums (their LDS words are the column sums', read by all by now)
  s_val = wave_sum_lane63(s_val);
  l1 = wave_sum_lane63(l1);
  __syncthreads();
  const int lane = t & (kWave - 1), wave = t / kWave;
  if (lane == kWave - 1) {
    s_v[wave] = s_val;
    s_v[4 + wave] = l1;
  }
  __syncthreads();
  if (t < 2) bsum[2 * b + t] = (s_v[4 * t] + s_v[4 * t + 1]) + (s_v[4 * t + 2] + s_v[4 * t + 3]);
}

__global__ __launch_bounds__(256) void ssim_bwd_kernel(const float* __restrict__ image,
                                                       const float* __restrict__ target, LossViews lv,
                                                       const float* __restrict__ dmap, int64_t map_stride,
                                                       float lambda, float* __restrict__ dL, int first) {
  __shared__ float4 s_v4[3 * kLH * kCols / 4];
  float* s_v = (float*)s_v4;
  const LossTile tl = loss_tile(lv, xcd_run(first + (int)blockIdx.x, lv.total_blocks));
  const LossView& q = lv.v[tl.view];
  const int W = q.W, H = q.H, t = threadIdx.x;
  const int64_t plane_px = (int64_t)W * H;
  const int64_t poff = 3 * q.pix_off + tl.plane * plane_px;
  const int x0 = tl.tx * q.tw, y0 = tl.ty * kLH;
  {
    const Column c = column_of(t, x0, y0, W);
    float d[3][kRows + 2 * kLR];
#pragma unroll
    for (int e = 0; e < 3; ++e) load_column(dmap + e * map_stride + poff, c, W, H, d[e]);
    const int row0 = (t / kCols) * kRows, col = t & (kCols - 1);
#pragma unroll
    for (int e = 0; e < 3; ++e)
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        float acc = lv.g[0] * d[e][r];
#pragma unroll
        for (int k = 1; k < kTaps; ++k) acc += lv.g[k] * d[e][r + k];
        s_v[(e * kLH + row0 + r) * kCols + col] = acc;
      }
  }
  __syncthreads();
  const float scale = 1.0f / ((float)lv.nviews * 3.0f * (float)plane_px);
  const int g = t & 31, px = x0 + kQ * g;
  const int m = kQ * g < q.tw ? (W - x0) - kQ * g : 0;  // (x0 + 4 g may pass the largest int: compare from below)
#pragma unroll 1
  for (int oy = t / 32; oy < kLH; oy += 8) {
    const int py = y0 + oy;
    if (m <= 0 || py >= H) continue;
    float f[3][kQ];
#pragma unroll
    for (int e = 0; e < 3; ++e) filter_row(s_v + (e * kLH + oy) * kCols, g, lv.g, f[e]);
    const int64_t pix = poff + (int64_t)py * W + px;
    const Quad x = load_quad(image + pix, m), y = load_quad(target + pix, m);
    Quad o;
#pragma unroll
    for (int p = 0; p < kQ; ++p) {
      const float dsdx = f[0][p] + 2.f * x[p] * f[1][p] + y[p] * f[2][p];
      const float sg = x[p] > y[p] ? 1.f : (x[p] < y[p] ? -1.f : 0.f);
      o[p] = ((1.0f - lambda) * sg - lambda * dsdx) * scale;
    }
    store_quad(dL + pix, m, o);
  }
}

// Per-view loss from its workgroups' sums: one workgroup per view, each thread
// a fixed stride of the sums in double, then a fixed tree.
__global__ __launch_bounds__(256) void loss_reduce_kernel(const float* __restrict__ bsum, LossViews lv,
                                                          float lambda, double* __restrict__ per_view,
                                                          float* __restrict__ loss) {
  __shared__ double s_s[256], s_l[256];
  const int v = blockIdx.x, t = threadIdx.x;
  const LossView& q = lv.v[v];
  const int nb = 3 * q.TX * q.TY;
  double s = 0.0, l1 = 0.0;
  for (int b = t; b < nb; b += 256) {
    s += (double)bsum[2 * (q.block_off + b) + 0];
    l1 += (double)bsum[2 * (q.block_off + b) + 1];
  }
  s_s[t] = s;
  s_l[t] = l1;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) {
      s_s[t] += s_s[t + o];
      s_l[t] += s_l[t + o];
    }
    __syncthreads();
  }
  if (t == 0) {
    const double n = 3.0 * (double)q.W * (double)q.H;
    const double lval = (1.0 - (double)lambda) * (s_l[0] / n) + (double)lambda * (1.0 - s_s[0] / n);
    per_view[v] = lval;
    loss[v] = (float)lval;
  }
}

// loss[V] = mean of the per-view losses, in view order.
__global__ void loss_mean_kernel(const double* __restrict__ per_view, int V, float* __restrict__ loss) {
  if (threadIdx.x != 0) return;
  double m = 0.0;
  for (int v = 0; v < V; ++v) m += per_view[v];
  loss[V] = (float)(m / V);
}

hipError_t launch_loss(const LossViews& lv, const float* image, const float* target, float lambda, float* loss,
                       float* dL, float* dmap, float* bsum, double* per_view, hipStream_t s) {
  const int nb = lv.total_blocks;
  if (nb == 0) return hipSuccess;
  const LossView& last = lv.v[lv.nviews - 1];
  const int64_t map_stride = 3 * (last.pix_off + (int64_t)last.W * last.H);  // floats of a map's plane
  image_launches(nb, [&](int first, dim3 grid) {
    hipLaunchKernelGGL(ssim_fwd_kernel, grid, dim3(256), 0, s, image, target, lv, dmap, map_stride, bsum, first);
  });
  if (dL)
    image_launches(nb, [&](int first, dim3 grid) {
      hipLaunchKernelGGL(ssim_bwd_kernel, grid, dim3(256), 0, s, image, target, lv, dmap, map_stride, lambda, dL, first);
    });
  if (loss) {
    hipLaunchKernelGGL(loss_reduce_kernel, dim3((unsigned)lv.nviews), dim3(256), 0, s, bsum, lv, lambda, per_view, loss);
    hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(64), 0, s, per_view, lv.nviews, loss);
  }
  return hipGetLastError();
}

}  // namespace gs

namespace gs {

// Mask terms of Eq. 7: lambda_m mean sigmoid(m) + lambda_sh mean sum_l w_l
// sigmoid(m^l), w_l = (2l + 1) / sum (2l' + 1) over bands 1..deg (each band
// weighted by its coefficient count, Sec. 3.2.3).  One thread per Gaussian:
// gradients accumulated (+=) into the mask-logit gradients; per-workgroup sums
// in a fixed order; a one-workgroup kernel adds them in double.
__global__ __launch_bounds__(256) void mask_loss_kernel(const float* __restrict__ m, const float* __restrict__ msh,
                                                        int64_t n, int deg, float lam_m, float lam_sh,
                                                        float* __restrict__ gm, float* __restrict__ gsh,
                                                        float* __restrict__ bsum) {
  __shared__ float s_red[2][4];
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  float a = 0.f, b = 0.f;
  if (i < n) {
    const float inv_n = 1.0f / (float)n;
    if (m) {
      const float s = 1.0f / (1.0f + __expf(-m[i]));
      a = s;
      if (gm) gm[i] += lam_m * s * (1.0f - s) * inv_n;
    }
    if (msh && deg > 0) {
      const float wsum = (float)(deg * (deg + 2));  // sum_{l=1..deg} (2l + 1)
      for (int l = 1; l <= deg; ++l) {
        const float w = (float)(2 * l + 1) / wsum;
        const float s = 1.0f / (1.0f + __expf(-msh[(int64_t)(l - 1) * n + i]));
        b += w * s;
        if (gsh) gsh[(int64_t)(l - 1) * n + i] += lam_sh * w * s * (1.0f - s) * inv_n;
      }
    }
  }
  a = wave_sum_lane63(a);
  b = wave_sum_lane63(b);
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (lane == kWave - 1) {
    s_red[0][wave] = a;
    s_red[1][wave] = b;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    bsum[2 * blockIdx.x + 0] = ((s_red[0][0] + s_red[0][1]) + s_red[0][2]) + s_red[0][3];
    bsum[2 * blockIdx.x + 1] = ((s_red[1][0] + s_red[1][1]) + s_red[1][2]) + s_red[1][3];
  }
}

__global__ __launch_bounds__(256) void mask_loss_reduce_kernel(const float* __restrict__ bsum, int nb, int64_t n,
                                                               float lam_m, float lam_sh, float* __restrict__ loss) {
  __shared__ double s_a[256], s_b[256];
  const int t = threadIdx.x;
  double a = 0.0, b = 0.0;
  for (int k = t; k < nb; k += 256) {
    a += (double)bsum[2 * k + 0];
    b += (double)bsum[2 * k + 1];
  }
  s_a[t] = a;
  s_b[t] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) {
      s_a[t] += s_a[t + o];
      s_b[t] += s_b[t + o];
    }
    __syncthreads();
  }
  if (t == 0) loss[0] = (float)((double)lam_m * s_a[0] / (double)n + (double)lam_sh * s_b[0] / (double)n);
}

hipError_t launch_mask_loss(const float* m, const float* msh, int64_t n, int deg, float lam_m, float lam_sh,
                            float* gm, float* gsh, float* loss, float* bsum, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int nb = (int)((n + 255) / 256);
  hipLaunchKernelGGL(mask_loss_kernel, dim3((unsigned)nb), dim3(256), 0, s, m, msh, n, deg, lam_m, lam_sh, gm, gsh,
                     bsum);
  if (loss) hipLaunchKernelGGL(mask_loss_reduce_kernel, dim3(1), dim3(256), 0, s, bsum, nb, n, lam_m, lam_sh, loss);
  return hipGetLastError();
}

// Four elements a thread: dL = scale_v (image - target), v the element's view.
// Bound by HBM: one 4-byte load of each image a thread moved the 111 MB of eight
// views of 3.09 Mpix in 32 us, 16-byte ones in 20.
__global__ __launch_bounds__(256) void l2_grad_kernel(const float* __restrict__ image,
                                                      const float* __restrict__ target, float* __restrict__ dL,
                                                      L2Args a) {
  const int64_t e = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  const int64_t total = a.end[a.nviews - 1];
  if (e >= total) return;
  int v = 0;
  while (e >= a.end[v]) ++v;
  if (e + 4 <= a.end[v]) {
    const Quad x = *(const Quad*)(image + e), y = *(const Quad*)(target + e);
    const float s = a.scale[v];
    *(Quad*)(dL + e) = Quad{s * (x.x - y.x), s * (x.y - y.y), s * (x.z - y.z), s * (x.w - y.w)};
  } else {  // the end of a view
    for (int64_t k = e; k < min(e + 4, total); ++k) {
      while (k >= a.end[v]) ++v;
      dL[k] = a.scale[v] * (image[k] - target[k]);
    }
  }
}

hipError_t launch_l2_grad(const float* image, const float* target, float* dL, const L2Args& a, hipStream_t s) {
  const int64_t total = a.nviews > 0 ? a.end[a.nviews - 1] : 0;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(l2_grad_kernel, dim3((unsigned)((total + 1023) / 1024)), dim3(256), 0, s, image, target, dL, a);
  return hipGetLastError();
}

}  // namespace gs
