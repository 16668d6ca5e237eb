// Target images for progressive training (Sec. 3.2.4): Gaussian blur with a
// shrinking kernel and area resampling to the current training resolution
// (Eq. 6).  Both act on every view of a call ([3][H][W] planes, views
// concatenated) and run when the schedule changes, not every step.
//
// Blur: filters columns, then rows, with the k normalised taps (k = 2 r + 1 <=
// 31), reflected about the edge pixels (index -1 reads 1).  A workgroup per
// (view, plane, tile of 128 - 2 r columns, rounded down to whole quads, x 16
// rows): a thread loads its column's 8 + 2 r values into registers, leaves 8
// column sums in LDS and filters rows from there, 4 neighbouring pixels from
// 16-byte reads.  One kernel per radius, so that taps and values stay in
// registers.  (From an LDS tile of 16 x 16 and its halo, a read per tap, the
// 5.9 M values of three views took 55 us at k = 7; now 13.)
//
// Resize: every output value averages the input over its box
// [x' W / W', (x' + 1) W / W') x [y' H / H', (y' + 1) H / H').  Overlaps
// are integers in units of 1 / W' (1 / H'), so the weights are exact; the sum
// is divided by W H once.  Two kernels (the rule and its figures: resize_by_box
// in gs_api.hip).  Boxes of few pixels, and narrow outputs: a thread per output
// value walks its box.  Large boxes, where such threads would be few, each with
// a long chain of loads W / W' columns apart: a workgroup takes a stretch of one
// output row whose boxes cover about 1000 input columns; its threads sum the
// box's rows per input column, side by side in memory, into LDS, then each
// output value adds its columns (three views of 5.9 M values to an eighth 18 ->
// 11 us; at a half or full size 1.3 to 1.5 times as slow as by box, and 5 to 50
// times for rows of 64 to 3 pixels).
#include "gs_common.h"
#include "kernels.h"

namespace gs {

typedef float Quad __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any float's address

// Position i reflected about 0 and n - 1 (unsigned: the period passes the
// largest int from n = 2^30 + 2 on).
__device__ __forceinline__ int64_t mirror_index(int64_t i, int n) {
  if (n == 1) return 0;
  const uint32_t p = 2u * (uint32_t)(n - 1), k = (uint32_t)(i < 0 ? -i : i) % p;  // even about 0
  return k < (uint32_t)n ? k : p - k;
}

template <int R>
__global__ __launch_bounds__(256) void blur_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                   BlurArgs b, int first) {
  constexpr int kCols = 128, kRows = kBlurTileH / 2, kQ = 4;
  constexpr int kTW = blur_tile_w(R);                     // output columns
  constexpr int kHalo = (2 * R + kQ - 1) / kQ * kQ;       // the row pass reads whole quads
  static_assert(kTW + kHalo <= kCols && kTW / kQ <= 32, "tile width");
  __shared__ float4 s_v4[kBlurTileH * kCols / 4];
  float* s_v = (float*)s_v4;
  const LossTile tl = loss_tile(b.views, first + (int)blockIdx.x);
  const LossView& q = b.views.v[tl.view];
  const int W = q.W, H = q.H, t = threadIdx.x;
  const int64_t poff = 3 * q.pix_off + tl.plane * (int64_t)W * H;
  const int x0 = tl.tx * q.tw, y0 = tl.ty * kBlurTileH;
  {  // column pass: thread t's column of the window, rows (t / 128) * 8 .. + 8
    const int col = t & (kCols - 1), row0 = __builtin_amdgcn_readfirstlane(t / kCols) * kRows;
    const float* src = in + poff + mirror_index((int64_t)x0 - R + col, W);
    float v[kRows + 2 * R];
    const int64_t ya = (int64_t)y0 + row0 - R;
    if (ya >= 0 && ya + kRows + 2 * R <= H) {  // no row of the wave's is reflected
#pragma unroll
      for (int i = 0; i < kRows + 2 * R; ++i) v[i] = src[(ya + i) * W];
    } else {
#pragma unroll
      for (int i = 0; i < kRows + 2 * R; ++i) v[i] = src[mirror_index(ya + i, H) * W];
    }
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) acc += b.g[k] * v[r + k];
      s_v[(row0 + r) * kCols + col] = acc;
    }
  }
  __syncthreads();
  // row pass: 8 rows of 32 threads, twice
  const int g = t & 31, px = x0 + kQ * g;
  const int m = kQ * g < q.tw ? (W - x0) - kQ * g : 0;  // (x0 + 4 g may pass the largest int: compare from below)
  for (int oy = t / 32; oy < kBlurTileH; oy += 8) {
    const int py = y0 + oy;
    if (m <= 0 || py >= H) continue;
    float v[kQ + kHalo];
#pragma unroll
    for (int k = 0; k < 1 + kHalo / kQ; ++k) {
      const float4 f = ((const float4*)(s_v + oy * kCols))[g + k];
      v[4 * k] = f.x, v[4 * k + 1] = f.y, v[4 * k + 2] = f.z, v[4 * k + 3] = f.w;
    }
    Quad o;
#pragma unroll
    for (int p = 0; p < kQ; ++p) {
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) acc += b.g[k] * v[p + k];
      o[p] = acc;
    }
    float* dst = out + poff + (int64_t)py * W + px;
    if (m >= kQ) {
      *(Quad*)dst = o;
    } else {
      dst[0] = o.x;
      if (m > 1) dst[1] = o.y;
      if (m > 2) dst[2] = o.z;
    }
  }
}

// a / b of non-negative numbers (in 32 bits where they fit: the 64-bit division
// is an order of magnitude longer).
__device__ __forceinline__ int64_t quotient(int64_t a, int64_t b) {
  return ((a | b) >> 32) == 0 ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}

// Units of 1 / no that input position i (of n) shares with output position o.
__device__ __forceinline__ float overlap(int64_t i, int64_t n, int64_t o, int64_t no) {
  return (float)(min((i + 1) * no, (o + 1) * n) - max(i * no, o * n));
}

__global__ __launch_bounds__(256) void resize_box_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                         ResizeArgs a) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.total_out) return;
  int v = 0;
  while (v + 1 < a.nviews && e >= 3 * a.v[v + 1].out_off) ++v;
  const ResizeView& q = a.v[v];
  const int64_t plane_out = (int64_t)q.Wo * q.Ho;
  const int64_t le = e - 3 * q.out_off;
  const int c = (int)(le / plane_out);
  const int64_t p = le - c * plane_out;
  const int yo = (int)(p / q.Wo), xo = (int)(p - (int64_t)yo * q.Wo);
  const int W = q.W, H = q.H, Wo = q.Wo, Ho = q.Ho;
  // input pixels whose box overlaps output pixel (xo, yo)
  const int xa = (int)(((int64_t)xo * W) / Wo), xb = (int)(((int64_t)(xo + 1) * W + Wo - 1) / Wo);
  const int ya = (int)(((int64_t)yo * H) / Ho), yb = (int)(((int64_t)(yo + 1) * H + Ho - 1) / Ho);
  const float* src = in + 3 * q.in_off + c * (int64_t)W * H;
  float acc = 0.f;
  for (int y = ya; y < yb; ++y) {
    float row = 0.f;
    for (int x = xa; x < xb; ++x) row += overlap(x, W, xo, Wo) * src[(int64_t)y * W + x];
    acc += overlap(y, H, yo, Ho) * row;
  }
  out[e] = acc * q.inv_area;
}

__global__ __launch_bounds__(256) void resize_kernel(const float* __restrict__ in, float* __restrict__ out,
                                                     ResizeArgs a) {
  __shared__ float4 s_col4[kResizeCols / 4];
  float* s_col = (float*)s_col4;
  const int t = threadIdx.x;
  for (int64_t item = blockIdx.x; item < a.items; item += gridDim.x) {
    int v = 0;
    while (v + 1 < a.nviews && item >= a.v[v + 1].item_off) ++v;
    const ResizeView& q = a.v[v];
    const int W = q.W, H = q.H, Wo = q.Wo, Ho = q.Ho;
    const int64_t li = item - q.item_off;
    const int64_t row = quotient(li, q.nseg);  // of the three planes' output rows
    const int c = row < Ho ? 0 : row < 2 * (int64_t)Ho ? 1 : 2;
    const int yo = (int)(row - c * (int64_t)Ho);
    // the stretch's first output and their number: t < nout, since xo0 + t and
    // xo0 + seg may pass the largest int
    const int xo0 = (int)(li - row * q.nseg) * q.seg, nout = min(q.seg, Wo - xo0);
    const int64_t xo = (int64_t)xo0 + t;
    // input rows of output row yo, columns of the stretch's outputs and of xo
    const int ya = (int)quotient((int64_t)yo * H, Ho), yb = (int)quotient((int64_t)(yo + 1) * H + Ho - 1, Ho);
    const int sa = (int)quotient((int64_t)xo0 * W, Wo), sb = (int)quotient((int64_t)(xo0 + nout) * W + Wo - 1, Wo);
    const int64_t xa = quotient(xo * W, Wo), xb = quotient((xo + 1) * W + Wo - 1, Wo);
    const float* src = in + 3 * q.in_off + c * (int64_t)W * H;
    float acc = 0.f;
    for (int64_t x0 = sa; x0 < sb; x0 += kResizeCols) {  // more than once only if W > kResizeCols W'
      const int n = (int)min(sb - x0, (int64_t)kResizeCols);
      __syncthreads();
      for (int x = 4 * t; x < n; x += 4 * 256) {  // four columns a thread
        Quad col = {0.f, 0.f, 0.f, 0.f};
        const float* p = src + x0 + x;
        if (x + 4 <= n) {
#pragma unroll 4
          for (int y = ya; y < yb; ++y) col += overlap(y, H, yo, Ho) * *(const Quad*)(p + (int64_t)y * W);
        } else {
          for (int y = ya; y < yb; ++y)
            for (int k = 0; k < 3; ++k)
              if (x + k < n) col[k] += overlap(y, H, yo, Ho) * p[(int64_t)y * W + k];
        }
        s_col4[x / 4] = make_float4(col.x, col.y, col.z, col.w);
      }
      __syncthreads();
      if (t < nout)
        for (int64_t x = max(xa, x0); x < min(xb, x0 + n); ++x) acc += overlap(x, W, xo, Wo) * s_col[x - x0];
    }
    if (t < nout) out[3 * q.out_off + row * Wo + xo] = acc * q.inv_area;
  }
}

// The kernel of radius r among those of radius R and below.
template <int R>
static void blur_radius(const float* in, float* out, const BlurArgs& b, hipStream_t s) {
  if (b.r == R) {
    image_launches(b.views.total_blocks, [&](int first, dim3 grid) {
      hipLaunchKernelGGL(blur_kernel<R>, grid, dim3(256), 0, s, in, out, b, first);
    });
  } else if constexpr (R > 0) {
    blur_radius<R - 1>(in, out, b, s);
  }
}

hipError_t launch_blur(const float* in, float* out, const BlurArgs& b, hipStream_t s) {
  if (b.views.total_blocks == 0) return hipSuccess;
  blur_radius<kMaxBlurRadius>(in, out, b, s);
  return hipGetLastError();
}

hipError_t launch_resize(const float* in, float* out, const ResizeArgs& a, hipStream_t s) {
  if (a.items == 0) return hipSuccess;
  if (a.by_box) {
    hipLaunchKernelGGL(resize_box_kernel, dim3((unsigned)((a.total_out + 255) / 256)), dim3(256), 0, s, in, out, a);
    return hipGetLastError();
  }
  const int64_t grid = a.items < (1 << 20) ? a.items : (1 << 20);
  hipLaunchKernelGGL(resize_kernel, dim3((unsigned)grid), dim3(256), 0, s, in, out, a);
  return hipGetLastError();
}

}  // namespace gs
