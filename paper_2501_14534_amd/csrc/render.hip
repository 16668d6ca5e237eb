// Per-tile front-to-back compositing (Eq. 2) and its backward.
//
// One workgroup per tile (global tile ids span all views of the call),
// launched in the heaviest-first order gs_bin_sort writes when the caller
// asks for it; each wave of it owns one sub-tile of pixels.  The backward
// walks the tile's sorted list in batches of splat records that the
// workgroup gathers into LDS together; the forward's waves walk the list
// independently (no workgroup barrier), each staging groups of 64 records
// into its own LDS with the gathers issued two groups ahead.  Every lane
// walks the staged records for its pixel(s), reading each as a wave-uniform
// LDS broadcast.  No MFMA: the work per (pixel, splat) pair is ~20 VALU
// operations and one exp.
//
// Sub-tile culling (CULL): while staging a batch, each record's conservative
// alpha >= 1/255 footprint (the ellipse q <= 2 ln(255 o'), widened by
// rounding margins) is tested against the live-pixel box of every 64-pixel
// block (a wave has one block per pixel of a thread): its bounding box first,
// then the ellipse itself (the minimum of q over the box); each wave then walks
// only the records whose bits it holds, taken from ballots in scalar registers,
// and of those only the blocks that they reach.  Culled records fail a
// per-pixel test for every pixel of that block, so the result is unchanged.
//
// Both walks are bound by vector issue where tiles are large (6M Gaussians,
// eight views up to 1080p, 32 x 32 tiles at 4 pixels a thread: 0.9 and 1.0 of
// the issue rate; the records that a 16 x 16 sub-tile walks reach 2.5 of its 4
// blocks, and composite in 34 of a block's 64 lanes).  Skipping blocks, keeping
// every decision in scalar masks and selecting lanes through the exec mask took
// the forward there from 1.75 to 1.36 ms and the backward from 3.30 to 2.59 ms;
// at 1M Gaussians, 1600 x 1064, 32 x 16 tiles at 2, from 0.231 to 0.197 and
// from 0.424 to 0.407 ms; with one block a wave (16 x 16 tiles, the same
// scene's forward) from 0.217 to 0.191 ms.
//
// Forward: lanes whose pixels have terminated drop out of the walk through
// the exec mask, and a wave leaves once all its pixels are done; the
// backward's waves vote before each batch and the workgroup leaves once every
// pixel is done.  At one pixel a thread the forward evaluates four records
// together and checks once whether a pixel stops among them: its deepest
// lists are walked by lone waves, bound by the latency of one record's chain
// (LDS read, exponential, decisions) and of one slice's gather.  With the four
// records' reads issued together, the transmittance as a plain chain of
// products and the gathers two slices ahead, the same image took 0.421 ->
// 0.385 ms for eight views of 1M Gaussians, 0.207 -> 0.175 for lists of 6000
// entries among 30K, 0.064 -> 0.058 at 200K, 0.021 -> 0.018 at 2K, and the
// hit counts of the eight views 0.428 -> 0.364.  (Eight records together, or
// slices further ahead, gain nothing: the registers cost a wave per SIMD.)
// Long lists can be split into forward chunks walked in parallel
// (a product pass gives each chunk its starting transmittance; see
// render_fwd_kernel), which shortens the critical path of the deepest tiles.
//
// Backward: the list is re-walked back to front from the tile's largest
// last_contrib; each pixel recovers the transmittance in front of a splat by
// dividing by (1 - alpha) and carries the dL/dC-weighted colour behind it, so
// no per-pixel list is stored.  Per-pair partials (9 floats) are summed over
// the lane's pixels, over the wave (a butterfly reduce-scatter over cross-lane
// swaps: 43 instructions for the 18 sums of two records), then over the workgroup's
// waves in a fixed order (LDS), and stored once per (tile, splat) at the
// pair's emission position: no atomics, so the result is bitwise reproducible.
#include "gs_common.h"
#include "kernels.h"

#include <type_traits>

namespace gs {

struct TileCtx {
  int view;
  int tx, ty;
  uint32_t start, end;
};

__device__ __forceinline__ TileCtx tile_ctx(const ViewTable& vt, const RenderArgs& a, int gtile) {
  TileCtx c;
  c.view = view_of_tile(vt, gtile);
  const ViewArgs& va = vt.v[c.view];
  const int lt = gtile - va.tile_off;
  c.ty = lt / va.TX;
  c.tx = lt - c.ty * va.TX;
  c.start = 0;
  c.end = 0;
  if (*a.status == 0) {
    c.start = a.ranges[2 * gtile];
    c.end = a.ranges[2 * gtile + 1];
  }
  return c;
}

// Pixels of a tile are split into one sub-tile per wave (as square as the
// tile allows, chosen on the host), and a sub-tile into PPT blocks of 64
// pixels (as square as it allows: 8 x 8 for the usual tiles).  A lane covers
// one pixel of each block, so that a wave can skip a block that a record does
// not reach.  Pixel p of thread t:
__device__ __forceinline__ void pixel_of(const RenderArgs& a, int t, int p, int tx, int ty, int* x, int* y) {
  const int w = t >> 6, l = t & (kWave - 1);
  const int sxi = w & ((1 << a.log2_sx) - 1), syi = w >> a.log2_sx;
  const int bxi = p & ((1 << a.log2_bx) - 1), byi = p >> a.log2_bx;
  *x = (tx << a.log2_tw) + (sxi << a.log2_sw) + (bxi << a.log2_bw) + (l & ((1 << a.log2_bw) - 1));
  *y = (ty << a.log2_th) + (syi << a.log2_sh) + (byi << (6 - a.log2_bw)) + (l >> a.log2_bw);
}

// Index of pixel p of this thread in the per-tile arrays of the workspace
// (consecutive threads next to each other).
__device__ __forceinline__ int tile_pixel(int p) { return p * (int)blockDim.x + (int)threadIdx.x; }

// Box of pixel centres [x0, x1] x [y0, y1]; empty when x0 > x1.
struct Box {
  float x0, x1, y0, y1;
};

// Box of the pixel centres of a block's live pixels (those that may still
// composite or receive gradient), the same value in every lane; empty when
// none is live.  Culling against it instead of the whole block drops the
// records that can only reach pixels that have already stopped.  `m`: the live
// lanes; (ox, oy): the block's first pixel centre, the same in every lane.
// Rows and columns come from the ballot by scalar bit operations, beside the
// vector units.
__device__ __forceinline__ Box live_box(uint64_t m, int log2_bw, float ox, float oy) {
  if (m == 0) return Box{__builtin_inff(), -__builtin_inff(), __builtin_inff(), -__builtin_inff()};
  uint64_t c = m;  // the rows folded into the first
  for (int s = 32; s >> log2_bw; s >>= 1) c |= c >> s;
  if (log2_bw < 6) c &= (1ull << (1 << log2_bw)) - 1;
  Box b;
  b.x0 = ox + (float)__builtin_ctzll(c);
  b.x1 = ox + (float)(63 - __builtin_clzll(c));
  b.y0 = oy + (float)(__builtin_ctzll(m) >> log2_bw);
  b.y1 = oy + (float)((63 - __builtin_clzll(m)) >> log2_bw);
  return b;
}

__device__ __forceinline__ float first_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

// Minimum over the box dx in [X0, X1], dy in [Y0, Y1] (relative to the
// centre) of q = A dx^2 + 2 B dx dy + C dy^2, positive definite: 0 when the
// centre is inside, else on an edge, where the 1-D minimiser is clamped to
// the edge (iA = 1 / A, iC = 1 / C).
__device__ __forceinline__ float qmin_box(float A, float B, float C, float iA, float iC, float X0, float X1,
                                          float Y0, float Y1) {
  if (X0 <= 0.f && X1 >= 0.f && Y0 <= 0.f && Y1 >= 0.f) return 0.f;
  auto qv = [&](float dx, float dy) { return A * dx * dx + 2.0f * B * dx * dy + C * dy * dy; };
  const float dyx0 = fminf(fmaxf(-B * X0 * iC, Y0), Y1), dyx1 = fminf(fmaxf(-B * X1 * iC, Y0), Y1);
  const float dxy0 = fminf(fmaxf(-B * Y0 * iA, X0), X1), dxy1 = fminf(fmaxf(-B * Y1 * iA, X0), X1);
  return fminf(fminf(qv(X0, dyx0), qv(X1, dyx1)), fminf(qv(dxy0, Y0), qv(dxy1, Y1)));
}

// Bit w set when record (u, v, conic, o', radius) may composite some pixel in
// box w of nboxes.
// Hardware reciprocals, roots and logarithms (a few units in the last place)
// are far inside the margins; where one overflows, the square decides.
__device__ __forceinline__ uint32_t footprint_mask(float4 ra, float4 rb, int nboxes, const Box* boxes) {
  const float u = ra.x, v = ra.y, A = ra.z, B = ra.w, C = rb.x, o = rb.y, r = rb.z;
  if (!(o >= kAlphaMin * 0.999f)) return 0u;  // alpha <= o' < 1/255 at every pixel
  float ex = r, ey = r, qm = 0.f, iA = 0.f, iC = 0.f;
  bool exact = false;
  const float det = A * C - B * B;
  if (det > 0.f) {
    const float tr = 0.5f * (A + C);
    const float lmax = tr + __builtin_amdgcn_sqrtf(fmaxf(0.f, tr * tr - det));
    if (lmax * lmax <= 1e3f * det) {  // condition number <= 1e3: rounding of q stays far below the margins
      // 2 ln(255 o') = 2 ln 2 (log2 255 + log2 o')
      qm = (2.0f * 0.69314718f * 1.002f) * (7.99435344f + __builtin_amdgcn_logf(o)) + 0.002f;
      const float k = fmaxf(qm, 0.f) * __builtin_amdgcn_rcpf(det);
      ex = fminf(r, __builtin_amdgcn_sqrtf(k * C) * 1.001f + 0.01f);
      ey = fminf(r, __builtin_amdgcn_sqrtf(k * A) * 1.001f + 0.01f);
      iA = __builtin_amdgcn_rcpf(A);
      iC = __builtin_amdgcn_rcpf(C);
      exact = true;
    }
  }
  ex += 0.5f;
  ey += 0.5f;
  uint32_t m = 0u;
#pragma unroll
  for (int w = 0; w < nboxes; ++w) {
    const Box b = boxes[w];
    bool hit = (u + ex >= b.x0) && (u - ex <= b.x1) && (v + ey >= b.y0) && (v - ey <= b.y1);
    // the ellipse q <= qm against the box of pixel centres (widened by 1e-3 px):
    // its bounding box can reach a corner of the box that the ellipse misses
    if (hit && exact)
      hit = qmin_box(A, B, C, iA, iC, b.x0 - 1e-3f - u, b.x1 + 1e-3f - u, b.y0 - 1e-3f - v, b.y1 + 1e-3f - v) <= qm;
    m |= hit ? (1u << w) : 0u;
  }
  return m;
}

// Entry selection.  Once a batch is staged, lane l of wave w reads the
// footprint mask of entry 64c + l; ballot p is the set of entries of chunk c
// that reach block p of wave w, returned with their union.  The walk takes the
// set bits in order from scalar registers, so no per-wave index list is built,
// stored or read.
template <int PPT, bool CULL>
__device__ __forceinline__ uint64_t chunk_bits(const uint16_t* s_mask, int c, int cnt, int wave, int lane,
                                               uint64_t (&mp)[PPT]) {
  const int i = c * kWave + lane;
  uint32_t bits = i < cnt ? (1u << PPT) - 1u : 0u;
  if (CULL && bits) bits &= (uint32_t)s_mask[i] >> (wave * PPT);
  uint64_t m = 0;
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    mp[p] = __ballot((bits >> p) & 1u);
    m |= mp[p];
  }
  return m;
}

// Dynamic LDS of the blend kernels, sized by the batch depth B and the wave count W:
//   records 3 x B float4 | [bwd] W x B x 9 partial sums | [bwd] B pair indices | B masks | [bwd] B rows
struct Lds {
  float4 *a, *b, *c;
  uint32_t* e;
  float* part;
  uint16_t* mask;
  uint16_t* row;
};

// Partial sums, in whole float4.
__host__ __device__ inline size_t part_bytes(int batch, int nwaves) {
  return (4 * (size_t)GS_GRAD_FLOATS * nwaves * batch + 15) & ~(size_t)15;
}

__host__ __device__ inline size_t lds_bytes(int batch, int nwaves, bool bwd) {
  size_t o = 3 * 16 * (size_t)batch;
  if (bwd) o += part_bytes(batch, nwaves) + 4 * (size_t)batch + 2 * (size_t)batch;
  o += 2 * (size_t)batch;
  return (o + 15) & ~(size_t)15;
}

__device__ inline Lds lds_carve(unsigned char* base, int batch, int nwaves, bool bwd) {
  Lds l;
  size_t o = 0;
  l.a = (float4*)(base + o), o += 16 * (size_t)batch;
  l.b = (float4*)(base + o), o += 16 * (size_t)batch;
  l.c = (float4*)(base + o), o += 16 * (size_t)batch;
  l.e = nullptr;
  l.part = nullptr;
  if (bwd) {
    l.part = (float*)(base + o), o += part_bytes(batch, nwaves);
    l.e = (uint32_t*)(base + o), o += 4 * (size_t)batch;
  }
  l.mask = (uint16_t*)(base + o), o += 2 * (size_t)batch;
  l.row = (uint16_t*)(base + o);
  return l;
}

// Largest backward batch: the partial sums of all waves stay within 18 KB.
__host__ __device__ inline int bwd_batch(int batch, int nwaves) {
  const int cap = 512 / nwaves;
  return batch < cap ? batch : cap;
}

__device__ __forceinline__ int tile_of_block(const RenderArgs& a) {
  return a.order ? (int)a.order[blockIdx.x] : (int)blockIdx.x;
}

// Whether this lane's bit is set in a wave mask.
__device__ __forceinline__ bool lane_in(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }
// The lanes whose pixel lies in the square of radius `rad` about an evaluated
// splat.  Decisions are kept as wave masks in scalar registers: they are
// combined beside the vector units and select lanes through the exec mask.
__device__ __forceinline__ uint64_t lanes_inside(const Eval& e, float rad) {
  return __ballot(fabsf(e.dx) <= rad) & __ballot(fabsf(e.dy) <= rad);
}

// Cross-lane moves of the backward's reduce-scatter.  permlane32_swap
// exchanges the upper 32 lanes of its first operand with the lower 32 lanes
// of its second, permlane16_swap the odd 16-lane rows of the first with the
// even rows of the second (both new on gfx950).  The pair result is read
// through a 64-bit cast.
__device__ __forceinline__ void swap_halves(float& a, float& b) {
  const uint64_t r = __builtin_bit_cast(
      uint64_t, __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                 false, false));
  a = __builtin_bit_cast(float, (uint32_t)r);
  b = __builtin_bit_cast(float, (uint32_t)(r >> 32));
}

__device__ __forceinline__ void swap_rows(float& a, float& b) {
  const uint64_t r = __builtin_bit_cast(
      uint64_t, __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b),
                                                 false, false));
  a = __builtin_bit_cast(float, (uint32_t)r);
  b = __builtin_bit_cast(float, (uint32_t)(r >> 32));
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}

// Sums each of 9 per-lane values of two records, x and y, over the 64 lanes of
// the wave (butterfly reduce-scatter: every step halves the values a lane
// carries).  The first step folds the halves of x into lanes 0-31 and those of y
// into lanes 32-63.  Element e = k + 5 b4 of the half's record ends in the two
// lanes of each (b5, b4, b3, b2, b1) with k: 0: (0, 0, 0), 1: (0, 0, 1),
// 2: (0, 1, 0), 3: (1, 0, 0), 4: (1, 0, 1) by (b3, b2, b1).  The tree is fixed,
// so the sums are reproducible, and the same whatever shares the reduction.
// Needs every lane of the wave active.  43 operations for 18 sums; one record
// alone takes 31 for its 9, one dependent step after the other.
__device__ __forceinline__ float reduce_scatter9x2(const float (&x)[GS_GRAD_FLOATS], const float (&y)[GS_GRAD_FLOATS],
                                                   bool b1, bool b2, bool b3) {
  float h[GS_GRAD_FLOATS];  // lane bit 5
#pragma unroll
  for (int k = 0; k < GS_GRAD_FLOATS; ++k) {
    float lo = x[k], hi = y[k];
    swap_halves(lo, hi);
    h[k] = lo + hi;
  }
  float z[5];  // lane bit 4: h0-h4 stay in even rows, h5-h8 go to odd rows
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    float lo = h[k], hi = k + 5 < GS_GRAD_FLOATS ? h[k + 5] : 0.0f;
    swap_rows(lo, hi);
    z[k] = lo + hi;
  }
  float t[5];  // lane bit 3
#pragma unroll
  for (int k = 0; k < 5; ++k) t[k] = z[k] + dpp_f<0x140>(z[k]);
  const float w0 = b3 ? t[3] : t[0], w1 = b3 ? t[4] : t[1], w2 = t[2];
  const float u0 = w0 + dpp_f<0x141>(w0), u1 = w1 + dpp_f<0x141>(w1), u2 = w2 + dpp_f<0x141>(w2);  // lane bit 2
  float v0 = b2 ? u2 : u0, v1 = u1;
  v0 += dpp_f<0x4E>(v0);  // lane bit 1
  v1 += dpp_f<0x4E>(v1);
  float v = b1 ? v1 : v0;
  v += dpp_f<0xB1>(v);
  return v;
}

// Walk modes of the forward kernel.
//   kFull:  Eq. 2 over one forward chunk of a tile's list (the whole list when
//           forward chunking is off): the image, or the chunk's results.
//   kCount: the same walk, counting instead of blending: per Gaussian, the
//           number of pixels where it is composited (the ray hits of Eq. 4),
//           added to a.hits; no image, no chunk states.  Lane l keeps the count
//           of its wave's entry l and adds it to the Gaussian's global counter
//           once the slice is walked.
//   kTPass: the product of (1 - alpha) over the chunk's splats that pass the
//           skip and square tests, ignoring the stop rule (stopped once under
//           1e-4, where its value no longer matters).
//
// Forward chunking.  A list longer than F = 2^log2_fchunk entries is split
// into chunks [start + kF, start + (k+1)F).  Three launches: every tile's
// first chunk (the only launch without chunking), which also leaves each
// pixel's transmittance after it (0 if it stopped) as the product P_0; the
// product pass over chunks 1 .. m-2, for the pixels still going after chunk
// 0 only; the full walk of chunks 1 .. m-1.  Chunk k starts from T_in =
// P_0 ... P_{k-1}: a pixel whose product fell under 1e-4 stopped in an
// earlier chunk (T only decreases), and otherwise T_in is its transmittance.
// Each chunk of a long list stores its colour, final T and last index;
// fwd_combine_kernel adds them up.  The critical path of a deep tile becomes
// about three chunks instead of its whole list.
typedef float Vec4 __attribute__((ext_vector_type(4)));
typedef float Vec3 __attribute__((ext_vector_type(3)));
// A prefetched record's words as a value of their own.  The compiler would
// otherwise split them into loop-carried scalars, whose register copies wait
// for the loads that have just been issued.
template <typename V>
__device__ __forceinline__ V held(V v) {
  asm("" : "+v"(v));
  return v;
}
__device__ __forceinline__ Vec3 load3(const float4* p) {
  const float* f = (const float*)p;
  return Vec3{f[0], f[1], f[2]};
}

enum : int { kFull = 0, kCount = 1, kTPass = 2 };
// Slices of 64 entries whose records a forward walk has in flight (three while
// the counting walk, without colours, has the registers).
template <int MODE>
constexpr int fwd_ring() { return MODE == kCount ? 3 : 2; }
// Pixel abscissa of a pixel that has stopped, or lies outside the image: NaN,
// which no record's square holds (an infinite radius included), so the walk
// needs no flag per pixel.
constexpr float kStopped = __builtin_nanf("");
__device__ __forceinline__ bool stopped(float px) { return px != px; }
constexpr int kIlp = 4;     // records evaluated together by the forward walk at one pixel per thread

// Stores and loads of the values one work item hands to another within a
// launch (image, T_final, last_contrib, chunk states).  COH: agent-scope
// relaxed atomics, which go to the device's coherence point instead of a
// compute die's L2, so an item on another die sees them once the flag that
// follows them is seen, without a cache-wide writeback or invalidate.
template <bool COH, typename T>
__device__ __forceinline__ void put(T* p, T v) {
  if (COH)
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else
    *p = v;
}
template <bool COH>
__device__ __forceinline__ void put4(float4* p, float4 v) {
  float* f = (float*)p;
  put<COH>(f + 0, v.x);
  put<COH>(f + 1, v.y);
  put<COH>(f + 2, v.z);
  put<COH>(f + 3, v.w);
}
template <bool COH, typename T>
__device__ __forceinline__ T get(const T* p) {
  return COH ? __hip_atomic_load(const_cast<T*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : *p;
}
template <bool COH>
__device__ __forceinline__ float4 get4(const float4* p) {
  const float* f = (const float*)p;
  return make_float4(get<COH>(f + 0), get<COH>(f + 1), get<COH>(f + 2), get<COH>(f + 3));
}

// One work item of a forward walk.  s_rec: per wave, the staged slice
// of records (a, b, c).  Items [0, nfslots) are
// the forward chunks that start at a forward boundary (slot order); the rest
// are each tile's first chunk, in the tile schedule.  Counting walks have no
// chunk items.  Returns the largest last_contrib this thread stored (0 if none).
template <int PPT, bool CULL, int MODE, bool COH = false>
__device__ __forceinline__ int fwd_item(const RenderArgs& a, const ViewTable& vt, float* __restrict__ image,
                                         float* __restrict__ T_final, int32_t* __restrict__ last_out, int64_t item,
                                         float4 (*s_rec)[3][kWave]) {
  constexpr bool COUNT = MODE == kCount, TPASS = MODE == kTPass;
  const int lf = COUNT ? 31 : a.log2_fchunk;
  const int64_t nfs = COUNT ? 0 : a.nfslots;
  int gtile;
  bool first;
  if (item < nfs) {
    const uint32_t owner = a.fslot_owner[item];
    if (owner >= (uint32_t)vt.total_tiles) return 0;  // no boundary here (uniform)
    gtile = (int)owner;
    first = false;
  } else {
    const int b = (int)(item - nfs);
    gtile = a.order ? (int)a.order[b] : b;
    first = true;
  }
  const TileCtx tc = tile_ctx(vt, a, gtile);
  const uint64_t fmask = (1ull << lf) - 1;
  const uint64_t cs64 = first ? (uint64_t)tc.start : (((uint64_t)item << lf) | ((uint64_t)tc.start & fmask));
  if (!first && !(cs64 > (uint64_t)tc.start && cs64 < (uint64_t)tc.end)) return 0;  // a record not of this list
  const uint32_t cs = (uint32_t)cs64;
  const uint32_t ce = (uint32_t)min(cs64 + (1ull << lf), (uint64_t)tc.end);
  const uint32_t len = tc.end - tc.start;
  const uint32_t nfc = len == 0 ? 1u : (uint32_t)(((uint64_t)len + fmask) >> lf);  // forward chunks of the list
  const uint32_t kf = (uint32_t)((cs64 - tc.start) >> lf);                           // this chunk
  if (TPASS && (kf == 0 || kf + 1 == nfc)) return 0;  // chunk 0 leaves its own; the last one is not needed
  const ViewArgs& va = vt.v[tc.view];
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  float4* s_a = s_rec[wave][0];
  float4* s_b = s_rec[wave][1];
  float4* s_c = s_rec[wave][2];

  // C: colour composited so far (the image, summed in list order whatever
  // the tiling); S: colour composited since the last chunk boundary (kept
  // apart so that the colour after a boundary is a sum of non-negative
  // segments, accurate relative to itself)
  float px[PPT], py[PPT], T[PPT], C0[PPT], C1[PPT], C2[PPT], S0[PPT], S1[PPT], S2[PPT];
  float ox[PPT], oy[PPT];
  int last[PPT];
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    int x, y;
    pixel_of(a, threadIdx.x, p, tc.tx, tc.ty, &x, &y);
    px[p] = (float)x + 0.5f;
    py[p] = (float)y + 0.5f;
    T[p] = 1.0f;
    C0[p] = C1[p] = C2[p] = 0.0f;
    S0[p] = S1[p] = S2[p] = 0.0f;
    last[p] = 0;
    if (CULL) {  // lane 0 holds the block's first pixel
      ox[p] = first_lane(px[p]);
      oy[p] = first_lane(py[p]);
    }
    if (!(x < va.W && y < va.H)) px[p] = kStopped;
  }

  const int tpx = 1 << (a.log2_tw + a.log2_th);
  const int lc = (COUNT || TPASS) ? 31 : a.log2_chunk;  // counting and products record no chunk states
  // chunk k >= 1 starts from the product of the earlier chunks' products
  bool dead[PPT];
#pragma unroll
  for (int p = 0; p < PPT; ++p) dead[p] = false;
  if (MODE == kFull && kf > 0) {
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      float t = 1.0f;
      for (uint32_t j = 1; j <= kf; ++j)
        t *= a.fprod[(int64_t)(((uint64_t)tc.start + ((uint64_t)j << lf)) >> lf) * tpx + tile_pixel(p)];
      T[p] = t;
      dead[p] = !stopped(px[p]) && t < kTMin;
      if (dead[p]) px[p] = kStopped;
    }
  }
  if (TPASS) {  // only the pixels still going after chunk 0
    const float* p0 = a.fprod + (int64_t)(((uint64_t)tc.start + (1ull << lf)) >> lf) * tpx;
#pragma unroll
    for (int p = 0; p < PPT; ++p)
      if (p0[tile_pixel(p)] < kTMin) px[p] = kStopped;
  }
  int nbnd = 0;  // chunk boundaries this wave recorded (uniform in the wave)
  // first backward boundary this walk can record: the first multiple of 2^lc
  // (relative to the list start) at or after cs, never the list start
  uint64_t b0 = (uint64_t)tc.start + ((((uint64_t)cs - tc.start) + ((1ull << lc) - 1)) >> lc << lc);
  if (b0 == (uint64_t)tc.start) b0 += 1ull << lc;
  // Each wave walks its own sub-tile independently (no workgroup barrier), in
  // slices of 64 entries (fewer with a smaller batch_depth or chunk; a power of
  // two, so that slices never straddle a chunk boundary): lane l stages entry l
  // into the wave's LDS, with its culling bits for the wave's live box.  The
  // records of the next R slices are in flight in R register sets, refilled as
  // soon as they are staged, and their ids one ring further ahead: late in a
  // deep list most records are culled, and a slice's walk is much shorter than a
  // gather's latency.
  constexpr int R = fwd_ring<MODE>();
  const uint32_t G = 1u << min(min(6, 31 - __clz(a.batch)), min(lc, lf));  // entries of a slice
  uint32_t gs = cs;                              // the slice: [gs, gs + G)
  Vec4 qa[R];                  // records of the slices gs + k G (in turn): (u, v, a, b)
  Vec3 qb[R], qc[R];           // (c, o', radius) and the colour
  uint32_t rid[R], nid[R];     // their ids; the ids R slices further on
  // every lane loads: a lane past a slice's or the list's end takes an entry
  // that is never staged (a load under a lane condition leaves a merged value
  // whose register copy waits for the load)
  const uint32_t elast = tc.end - 1;  // used only when the walk has entries
#pragma unroll
  for (int k = 0; k < R; ++k) {
    qa[k] = Vec4{0.f, 0.f, 0.f, 0.f};
    qb[k] = qc[k] = Vec3{0.f, 0.f, 0.f};
    rid[k] = nid[k] = 0;
  }
  auto fetch = [&](int k) {
    const float4* rec = a.splats + (size_t)rid[k] * 3;
    qa[k] = *(const Vec4*)rec;
    qb[k] = load3(rec + 1);
    if (!COUNT) qc[k] = load3(rec + 2);
  };
  if (cs < ce) {
#pragma unroll
    for (int k = 0; k < R; ++k) rid[k] = a.ids[min(gs + k * G + lane, elast)];
    // issued in the order of the loop, so that its waits count on it
#pragma unroll
    for (int k = 0; k < R; ++k) {
      fetch(k);
      __builtin_amdgcn_sched_barrier(0);
      nid[k] = a.ids[min(gs + (R + k) * G + lane, elast)];
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // one slice from register set k
  uint32_t left = ce - cs;  // entries from gs on; 0: the walk is done
  Box box[PPT];
  uint64_t was_live[PPT];  // the pixels that the boxes hold
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    was_live[p] = 0;
    box[p] = live_box(0, 0, 0.f, 0.f);
  }
  auto walk_slice = [&](int k) {
    if (k == 0) {  // once a ring: what is still live, and where
      // (a box is made anew only when its pixels have changed: its chain of scalar
      // operations is a tenth of a deep list's slice, and four boxes of a 6M-Gaussian
      // step took 1.35 ms for 1.30)
      uint64_t alive = 0;
#pragma unroll
      for (int p = 0; p < PPT; ++p) {
        const uint64_t live = __ballot(!stopped(px[p]));
        alive |= live;
        if (CULL && live != was_live[p]) {  // uniform
          const Box b = live_box(live, a.log2_bw, ox[p], oy[p]);
          box[p] = PPT > 1 ? b : Box{first_lane(b.x0), first_lane(b.x1), first_lane(b.y0), first_lane(b.y1)};
        }
        was_live[p] = live;
      }
      if (alive == 0) left = 0;  // every pixel of this wave has stopped
    }
    const uint64_t rel = gs - tc.start;
    if (MODE == kFull && left != 0 && rel != 0 && (rel & ((1ull << lc) - 1)) == 0) {
      // a chunk boundary of the backward: record each pixel's transmittance
      // here and the colour of the chunk that ends here, then start a new chunk
      const int64_t slot = (int64_t)(gs >> lc);
      float4* st = a.state + slot * tpx;
#pragma unroll
      for (int p = 0; p < PPT; ++p) {
        put4<COH>(st + tile_pixel(p), make_float4(T[p], S0[p], S1[p], S2[p]));
        S0[p] = S1[p] = S2[p] = 0.0f;
      }
      if (lane == 0) a.slot_owner[slot] = (uint32_t)gtile;  // every wave that gets here writes the same
      ++nbnd;
    }
    const int cnt = (int)min(G, left);
    uint32_t bits = lane < cnt ? (1u << PPT) - 1u : 0u;  // the blocks that the entry may reach
    const Vec4 ha = held(qa[k]);
    const Vec3 hb = held(qb[k]);
    const float4 ra = make_float4(ha.x, ha.y, ha.z, ha.w), rb = make_float4(hb.x, hb.y, hb.z, 0.0f);
    if (bits) {
      s_a[lane] = staged_a(ra);
      *(Vec3*)(s_b + lane) = Vec3{kQScale * rb.x, rb.y, rb.z};
      if (!COUNT) {
        const Vec3 hc = held(qc[k]);
        *(Vec3*)(s_c + lane) = hc;
      }
      if (CULL) bits = footprint_mask(ra, rb, PPT, box);
    }
    const uint32_t gid = rid[k];
    rid[k] = nid[k];
    fetch(k);  // the slice R on, into the registers just staged from
    nid[k] = a.ids[min(gs + 2 * R * G + lane, elast)];
    wave_lds_sync();  // the staged slice is visible to the whole wave
    uint64_t mp[PPT], m = 0;  // the entries that reach block p, and their union
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      mp[p] = __ballot((bits >> p) & 1u);
      m |= mp[p];
    }
    if (m != 0) {
      const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
      const int idx0 = (int)(gs - tc.start) + 1;  // list position of the slice's entry 0, from 1
      uint32_t hits = 0;                          // COUNT: lane l's, the pixels that composite entry l
      if constexpr (PPT == 1) {
        // N records together (in list order).  Their falloff and alpha do not
        // depend on the transmittance, and neither do the lanes that use them
        // unless one stops within the group: with alpha 0 in the other lanes
        // the transmittance is a chain of N products, checked once at its end
        // (it only falls).  Only a group in which a pixel stops goes through the
        // records one by one, to find the lanes that take each.
        auto group = [&](auto size) {
          constexpr int N = decltype(size)::value;
          int jq[N];
          float4 ra[N], rb[N], rc[N];
          float al[N], Tq[N + 1];
          uint64_t use[N], any = 0;
#pragma unroll
          for (int q = 0; q < N; ++q) {
            jq[q] = __builtin_ctzll(m);
            m &= m - 1;
          }
#pragma unroll
          for (int q = 0; q < N; ++q) {
            ra[q] = s_a[jq[q]];
            rb[q] = s_b[jq[q]];
          }
          // all of the group's reads are in flight before the first is used
          __builtin_amdgcn_sched_barrier(0);
          Eval e[N];
#pragma unroll
          for (int q = 0; q < N; ++q)
            eval_splat_all(px[0], py[0], ra[q].x, ra[q].y, ra[q].z, ra[q].w, rb[q].x, rb[q].y, &e[q]);
#pragma unroll
          for (int q = 0; q < N; ++q) rc[q] = COUNT || TPASS ? zero4 : s_c[jq[q]];
#pragma unroll
          for (int q = 0; q < N; ++q) {
            al[q] = e[q].alpha;
            use[q] = lanes_inside(e[q], rb[q].z) & __ballot(!(al[q] < kAlphaMin));
            any |= use[q];
          }
          float am[N];  // alpha of the lanes that take the record, else 0
          Tq[0] = T[0];
#pragma unroll
          for (int q = 0; q < N; ++q) {
            am[q] = lane_in(use[q]) ? al[q] : 0.0f;
            Tq[q + 1] = Tq[q] * (1.0f - am[q]);
          }
          if ((any & __ballot(Tq[N] < kTMin)) != 0) {  // wave-uniform: some pixel stops here
            uint64_t gone = 0;
#pragma unroll
            for (int q = 0; q < N; ++q) {
              use[q] &= ~gone;
              const uint64_t low = use[q] & __ballot(Tq[q] * (1.0f - al[q]) < kTMin);
              gone |= low;                 // stop before this splat
              if (!TPASS) use[q] &= ~low;  // the product pass multiplies the stopping splat in as well
              am[q] = lane_in(use[q]) ? al[q] : 0.0f;
              Tq[q + 1] = Tq[q] * (1.0f - am[q]);
            }
            px[0] = lane_in(gone) ? kStopped : px[0];
          }
#pragma unroll
          for (int q = 0; q < N; ++q) {
            const float w = am[q] * Tq[q];
            C0[0] += rc[q].x * w;
            C1[0] += rc[q].y * w;
            C2[0] += rc[q].z * w;
            S0[0] += rc[q].x * w;
            S1[0] += rc[q].y * w;
            S2[0] += rc[q].z * w;
            last[0] = lane_in(use[q]) ? idx0 + jq[q] : last[0];
            if (COUNT) hits = lane_in(1ull << jq[q]) ? (uint32_t)__popcll(use[q]) : hits;
          }
          T[0] = Tq[N];
        };
        for (int n = __popcll(m); n >= kIlp; n -= kIlp) group(std::integral_constant<int, kIlp>());
        if (__popcll(m) >= 2) group(std::integral_constant<int, 2>());
        if (m != 0) group(std::integral_constant<int, 1>());
      } else {
        // one record at a time, over the blocks that it reaches (wave-uniform
        // branches).  A record's lanes are selected through the exec mask (three
        // vector operations fewer than by value).
        for (; m != 0; m &= m - 1) {
          const int j = __builtin_ctzll(m);
          const float4 ra = s_a[j], rb = s_b[j], rc = COUNT || TPASS ? zero4 : s_c[j];
          uint32_t taken = 0;
#pragma unroll
          for (int p = 0; p < PPT; ++p)
            if ((mp[p] >> j) & 1ull) {
              Eval e;
              eval_splat_all(px[p], py[p], ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, &e);
              const float Tn = T[p] * (1.0f - e.alpha);
              const uint64_t use = lanes_inside(e, rb.z) & __ballot(!(e.alpha < kAlphaMin));
              const uint64_t low = use & __ballot(Tn < kTMin);
              // the product pass multiplies the stopping splat in as well
              const uint64_t take = TPASS ? use : use & ~low;
              if (lane_in(take)) {
                const float w = e.alpha * T[p];
                C0[p] += rc.x * w;
                C1[p] += rc.y * w;
                C2[p] += rc.z * w;
                S0[p] += rc.x * w;
                S1[p] += rc.y * w;
                S2[p] += rc.z * w;
                T[p] = Tn;
                last[p] = idx0 + j;
              }
              px[p] = lane_in(low) ? kStopped : px[p];  // stop before this splat
              if (COUNT) taken += (uint32_t)__popcll(take);
            }
          if (COUNT) hits = lane_in(1ull << j) ? taken : hits;
        }
      }
      // the slice's counters: lane l adds entry l's hits to its Gaussian
      if (COUNT && hits != 0) atomicAdd(a.hits + ((int64_t)gid - (int64_t)tc.view * a.n), hits);
    }
    wave_lds_sync();  // every lane has read the slice before the next one overwrites it
    gs += G;
    left = left > G ? left - G : 0;
  };
  // (no way out between the steps: paths that skip a step's loads would make
  // the waits of all others wait for the newest load)
  while (left != 0) {
#pragma unroll
    for (int k = 0; k < R; ++k) walk_slice(k);
  }

  if (COUNT) return 0;
  if (TPASS) {  // the product, at the boundary that ends this chunk
    float* fp = a.fprod + (int64_t)((uint64_t)ce >> lf) * tpx;
#pragma unroll
    for (int p = 0; p < PPT; ++p) fp[tile_pixel(p)] = T[p];
    return 0;
  }
  // Each recorded state becomes (T there, colour composited after it within
  // this walk): the suffix sums of the segments' colours, last one first.  The
  // states are read kSuf at a time, all loads in flight together (a deep list
  // records dozens of states, and one load at a time would put as many memory
  // round trips on the walk's critical path).
  constexpr int kSuf = PPT >= 4 ? 1 : 4 / PPT;
  for (int k0 = nbnd - 1; k0 >= 0; k0 -= kSuf) {
    float4 v[kSuf][PPT];
#pragma unroll
    for (int i = 0; i < kSuf; ++i) {
      if (k0 - i < 0) break;  // wave-uniform
      const int64_t slot = (int64_t)((b0 + ((uint64_t)(k0 - i) << lc)) >> lc);
#pragma unroll
      for (int p = 0; p < PPT; ++p) v[i][p] = get4<COH>(a.state + slot * tpx + tile_pixel(p));
    }
#pragma unroll
    for (int i = 0; i < kSuf; ++i) {
      if (k0 - i < 0) break;
      const int64_t slot = (int64_t)((b0 + ((uint64_t)(k0 - i) << lc)) >> lc);
#pragma unroll
      for (int p = 0; p < PPT; ++p) {
        const float e0 = v[i][p].y, e1 = v[i][p].z, e2 = v[i][p].w;  // colour of the chunk before the boundary
        put4<COH>(a.state + slot * tpx + tile_pixel(p), make_float4(v[i][p].x, S0[p], S1[p], S2[p]));
        S0[p] = e0 + S0[p];
        S1[p] = e1 + S1[p];
        S2[p] = e2 + S2[p];
      }
    }
  }

  if (nfc > 1) {
    // one chunk of several: its colour, final T and last index (-1: the pixel
    // had stopped before the chunk), at the boundary that ends it, or for the
    // last chunk at the one that starts it (second half of the arrays); the
    // first chunk also leaves P_0 (0 for the pixels that stopped in it)
    const int64_t idx = kf + 1 < nfc ? (int64_t)((uint64_t)ce >> lf) : a.nfslots + (int64_t)((uint64_t)cs >> lf);
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      a.fres[idx * tpx + tile_pixel(p)] = make_float4(C0[p], C1[p], C2[p], T[p]);
      a.flast[idx * tpx + tile_pixel(p)] = dead[p] ? -1 : last[p];
      if (kf == 0) a.fprod[idx * tpx + tile_pixel(p)] = stopped(px[p]) ? 0.0f : T[p];
    }
    return 0;
  }
  const int64_t plane = (int64_t)va.W * va.H;
  int my_max = 0;
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    int x, y;
    pixel_of(a, threadIdx.x, p, tc.tx, tc.ty, &x, &y);
    if (x < va.W && y < va.H) {
      const int64_t pix = (int64_t)y * va.W + x;
      float* img = image + 3 * (int64_t)va.pix_off;
      put<COH>(img + pix, C0[p] + T[p] * a.bg[0]);
      put<COH>(img + plane + pix, C1[p] + T[p] * a.bg[1]);
      put<COH>(img + 2 * plane + pix, C2[p] + T[p] * a.bg[2]);
      put<COH>(T_final + va.pix_off + pix, T[p]);
      put<COH>(last_out + va.pix_off + pix, last[p]);
      my_max = max(my_max, last[p]);
    }
  }
  return my_max;
}

// Work items [item_base, item_base + gridDim.x) of a forward walk, one per workgroup.
// The kernel is held to 96, 80 and 128 registers at 1, 2 and 4 pixels a thread
// (five, six and four waves per SIMD).  At 1 it takes 94: held to 80 it spills 11,
// whose reloads wait for the gathers in flight (200K Gaussians 0.058 -> 0.062 ms).
// At 2 it spills one, outside of the walk's loop.
template <int PPT>
constexpr int fwd_waves() { return PPT == 1 ? 5 : PPT == 2 ? 6 : 4; }
template <int PPT, bool CULL, int MODE>
__global__ __launch_bounds__(256, fwd_waves<PPT>()) void render_fwd_kernel(RenderArgs a, ViewTable vt,
                                                                           float* __restrict__ image,
                                                                           float* __restrict__ T_final,
                                                                           int32_t* __restrict__ last_out,
                                                                           int64_t item_base) {
  __shared__ float4 s_rec[4][3][kWave];
  fwd_item<PPT, CULL, MODE>(a, vt, image, T_final, last_out, (int64_t)blockIdx.x + item_base, s_rec);
}

// Forward chunking: the tiles with several chunks.  Per pixel, the chunks'
// colours are added from the last one down (giving the colour composited
// from each forward boundary on, which the backward adds to its chunk
// states), the final T is the one of the last chunk the pixel entered alive,
// and the last index the largest.  One workgroup per tile, in the schedule.
template <int PPT>
__global__ __launch_bounds__(256) void fwd_combine_kernel(RenderArgs a, ViewTable vt, float* __restrict__ image,
                                                          float* __restrict__ T_final,
                                                          int32_t* __restrict__ last_out) {
  const int gtile = tile_of_block(a);
  const TileCtx tc = tile_ctx(vt, a, gtile);
  const int lf = a.log2_fchunk;
  const uint32_t len = tc.end - tc.start;
  const uint32_t nfc = (uint32_t)(((uint64_t)len + ((1ull << lf) - 1)) >> lf);
  if (nfc < 2) return;
  const ViewArgs& va = vt.v[tc.view];
  const int tpx = 1 << (a.log2_tw + a.log2_th);
  const int64_t plane = (int64_t)va.W * va.H;
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    int x, y;
    pixel_of(a, threadIdx.x, p, tc.tx, tc.ty, &x, &y);
    const int q = tile_pixel(p);
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, Tf = 1.f;
    bool have_T = false;
    int last = 0;
    for (int k = (int)nfc - 1; k >= 0; --k) {
      const uint64_t bk = (uint64_t)tc.start + ((uint64_t)k << lf);
      const int64_t idx = k + 1 < (int)nfc ? (int64_t)((bk + (1ull << lf)) >> lf) : a.nfslots + (int64_t)(bk >> lf);
      const float4 r = a.fres[idx * tpx + q];
      const int l = a.flast[idx * tpx + q];
      s0 = r.x + s0;
      s1 = r.y + s1;
      s2 = r.z + s2;
      if (k > 0) a.fsuf[(int64_t)(bk >> lf) * tpx + q] = make_float4(s0, s1, s2, 0.f);
      if (!have_T && l >= 0) {
        Tf = r.w;
        have_T = true;
      }
      last = max(last, l);
    }
    if (x < va.W && y < va.H) {
      const int64_t pix = (int64_t)y * va.W + x;
      float* img = image + 3 * (int64_t)va.pix_off;
      img[pix] = s0 + Tf * a.bg[0];
      img[plane + pix] = s1 + Tf * a.bg[1];
      img[2 * plane + pix] = s2 + Tf * a.bg[2];
      T_final[va.pix_off + pix] = Tf;
      last_out[va.pix_off + pix] = last;
    }
  }
}

// Owners of the forward boundaries: slot (start + kF) >> log2_fchunk of a
// tile's list, k >= 1.  One thread per tile.
__global__ void fwd_mark_kernel(RenderArgs a, int total_tiles) {
  const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gt >= total_tiles || *a.status != 0) return;
  const uint64_t start = a.ranges[2 * gt], end = a.ranges[2 * gt + 1];
  const int lf = a.log2_fchunk;
  for (uint64_t q = start + (1ull << lf); q < end; q += 1ull << lf) a.fslot_owner[q >> lf] = (uint32_t)gt;
}

constexpr float kPosScale = 2.77258872223978124f;  // 4 ln 2 = -2 / kQScale

// The loss gradient a backward walk reads: dL/dimage from memory, or (fused
// with the forward) the mean-squared-error gradient computed per pixel from
// the image the forward wrote and the target, dL = scale_v (image - target)
// in single precision, as gs_l2_grad computes it; the tile's first backward
// item also stores it when dL_out is given.
struct LossIn {
  const float* dL_dimage;
  const float* image;
  const float* target;
  float* dL_out;
  float scale[GS_MAX_VIEWS];
};

// One work item of the backward walk.  Items [0, nslots) are the chunks that
// start at a recorded boundary (slot order, so the long lists' chunks start
// first); the rest are each tile's first chunk, in the tile schedule.  smem:
// lds_bytes(bwd_batch(batch, waves), waves, true) bytes.  ok false (a wait for
// the tile's forward that timed out): the item's loss gradient is NaN.  walked
// >= 0: the tile's largest last_contrib, known beforehand.
template <int PPT, bool CULL, bool L2>
__device__ __forceinline__ void bwd_item(const RenderArgs& a, const ViewTable& vt, const float* __restrict__ T_final,
                                         const int32_t* __restrict__ last_in, const LossIn& loss,
                                         float* __restrict__ grad_pair, int64_t item, unsigned char* smem,
                                         bool ok = true, int walked = -1) {
  constexpr int kMaxChunks = 8;  // of 64 entries in a batch
  __shared__ int s_max[4];
  __shared__ Box s_box[4 * PPT];  // live box of every wave's blocks
  __shared__ uint64_t s_hit[kMaxChunks][4];  // entries of a chunk that a wave added to
  const int lg = a.log2_chunk;
  int gtile;
  bool first;
  if (item < a.nslots) {
    const uint32_t owner = a.slot_owner[item];
    if (owner >= (uint32_t)vt.total_tiles) return;  // no boundary here (uniform)
    gtile = (int)owner;
    first = false;
  } else {
    const int b = (int)(item - a.nslots);
    gtile = a.order ? (int)a.order[b] : b;
    first = true;
  }
  const TileCtx tc = tile_ctx(vt, a, gtile);
  const uint64_t cmask = (1ull << lg) - 1;
  // chunk [cs, ce) of the tile's list [start, end)
  const uint64_t cs = first ? (uint64_t)tc.start : (((uint64_t)item << lg) | ((uint64_t)tc.start & cmask));
  const uint64_t ce = min(cs + (1ull << lg), (uint64_t)tc.end);
  if (!first && !(cs > (uint64_t)tc.start && cs < (uint64_t)tc.end)) return;  // a record not of this list
  // a chunk at or past the tile's largest last_contrib has nothing to do (uniform)
  if (!first && walked >= 0 && cs >= (uint64_t)tc.start + (uint64_t)walked) return;
  const ViewArgs& va = vt.v[tc.view];
  const int nthreads = blockDim.x;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, nwaves = nthreads / kWave;
  const int64_t plane = (int64_t)va.W * va.H;
  const int batch = bwd_batch(a.batch, nwaves);
  const Lds L = lds_carve(smem, batch, nwaves, true);
  float4* s_a = L.a;
  float4* s_b = L.b;
  float4* s_c = L.c;
  uint32_t* s_e = L.e;
  float* s_part = L.part;  // per-wave partial sums of one batch: [nwaves][batch][9]
  uint16_t* s_mask = L.mask;

  // this lane's element of the reduce-scatter (see reduce_scatter9x2)
  const bool b1 = (lane >> 1) & 1, b2 = (lane >> 2) & 1, b3 = (lane >> 3) & 1;
  const int my_k = b3 ? (b1 ? 4 : 3) : b1 ? 1 : b2 ? 2 : 0, my_e = my_k + 5 * ((lane >> 4) & 1);
  const bool writer = (lane & 1) == 0 && !(b2 && (b1 || b3)) && my_e < GS_GRAD_FLOATS;
  // per element, the factor the walk leaves out: with m = -2 dL/dq,
  // dL/d(u, v) = (-2/k) dL/dq (A dx + B dy, B dx + C dy) = -(2 ln 2) m (a dx + b/2 dy, ...),
  // dL/d(A, B, C) = dL/dq (dx^2, 2 dx dy, dy^2) = -m (dx^2 / 2, dx dy, dy^2 / 2)
  const float escale = my_e < 2 ? -0.5f * kPosScale : my_e == 3 ? -1.0f : my_e < 5 ? -0.5f : 1.0f;

  float px[PPT], py[PPT], T[PPT], g0[PPT], g1[PPT], g2[PPT], RdL[PPT];
  int lc[PPT];
  int my_max = 0;
#pragma unroll
  for (int p = 0; p < PPT; ++p) {
    int x, y;
    pixel_of(a, threadIdx.x, p, tc.tx, tc.ty, &x, &y);
    px[p] = (float)x + 0.5f;
    py[p] = (float)y + 0.5f;
    T[p] = 1.0f;
    g0[p] = g1[p] = g2[p] = RdL[p] = 0.0f;
    lc[p] = 0;
    if (x < va.W && y < va.H) {
      const int64_t pix = (int64_t)y * va.W + x;
      const int64_t e0 = 3 * (int64_t)va.pix_off + pix;
      T[p] = get<L2>(T_final + va.pix_off + pix);
      lc[p] = get<L2>(last_in + va.pix_off + pix);
      if (L2) {
        const float sc = ok ? loss.scale[tc.view] : __builtin_nanf("");
        g0[p] = sc * (get<L2>(loss.image + e0) - loss.target[e0]);
        g1[p] = sc * (get<L2>(loss.image + e0 + plane) - loss.target[e0 + plane]);
        g2[p] = sc * (get<L2>(loss.image + e0 + 2 * plane) - loss.target[e0 + 2 * plane]);
        if (first && loss.dL_out) {
          loss.dL_out[e0] = g0[p];
          loss.dL_out[e0 + plane] = g1[p];
          loss.dL_out[e0 + 2 * plane] = g2[p];
        }
      } else {
        g0[p] = loss.dL_dimage[e0];
        g1[p] = loss.dL_dimage[e0 + plane];
        g2[p] = loss.dL_dimage[e0 + 2 * plane];
      }
      RdL[p] = T[p] * (a.bg[0] * g0[p] + a.bg[1] * g1[p] + a.bg[2] * g2[p]);
      my_max = max(my_max, lc[p]);
    }
  }
  // workgroup max of last_contrib
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) my_max = max(my_max, __shfl_xor(my_max, o, kWave));
  if (lane == 0) s_max[wave] = my_max;
  __syncthreads();
  int maxlast = 0;
  for (int w = 0; w < nwaves; ++w) maxlast = max(maxlast, s_max[w]);
  maxlast = min(maxlast, (int)(tc.end - tc.start));  // never walk past the tile's list
  const uint64_t wlim = (uint64_t)tc.start + (uint64_t)maxlast;

  // Pairs that no pixel composites receive no gradient: their rows are not
  // written and their live bytes stay 0 (cleared before the launch), so the
  // per-record sums skip them.  (About 4 in 5 pairs at 1M Gaussians lie behind
  // every pixel's last contributor: writing zero rows at their scattered
  // emission positions cost more than the rest of the walk's stores; half of the
  // others are culled or miss every pixel: leaving those out too took the walk
  // from 427 to 406 us and the sums from 95 to 81 at 1M Gaussians in eight
  // views, from 2590 to 2530 and from 490 to 421 at 6M.)  With a.zero_rows the
  // pairs in front of the last contributor get their rows all the same.

  // Starting state at the chunk's end: the final one when the walk ends in
  // this chunk, else the forward's record at ce (transmittance there, and the
  // colour composited after it, which gives the dL/dC-weighted colour behind)
  // for the pixels that still composite after ce; the others keep the final
  // state.  With forward chunking the record holds the colour composited
  // after ce within its forward chunk; the later chunks' colour is added.
  if (ce < wlim) {
    const int tpx = 1 << (a.log2_tw + a.log2_th);
    const float4* st = a.state + (int64_t)(ce >> lg) * tpx;
    const float4* sf = nullptr;
    if (a.log2_fchunk < 31) {
      const int lf = a.log2_fchunk;
      const uint64_t nxt = (uint64_t)tc.start + ((((ce - tc.start) >> lf) + 1) << lf);  // next forward boundary
      if (nxt < (uint64_t)tc.end) sf = a.fsuf + (int64_t)(nxt >> lf) * tpx;
    }
    const int rel = (int)(ce - tc.start);
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
      if (lc[p] > rel) {
        const float4 v = get4<L2>(st + tile_pixel(p));
        float c0 = v.y, c1 = v.z, c2 = v.w;
        if (sf) {
          const float4 w = sf[tile_pixel(p)];
          c0 += w.x;
          c1 += w.y;
          c2 += w.z;
        }
        T[p] = v.x;
        RdL[p] = RdL[p] + (c0 * g0[p] + c1 * g1[p] + c2 * g2[p]);
      }
    }
  }

  const uint32_t cstart = (uint32_t)cs;
  const uint32_t wend = (uint32_t)min(ce, wlim);
  for (uint32_t be = wend; be > cstart;) {
    const uint32_t bs = (be - cstart > (uint32_t)batch) ? be - batch : cstart;
    const int cnt = (int)(be - bs);
    if (CULL) {
      // live pixels: those with an entry of this batch before their last contributor
#pragma unroll
      for (int p = 0; p < PPT; ++p) {
        const uint64_t live = __ballot(lc[p] > (int)(bs - tc.start));
        const Box b = live_box(live, a.log2_bw, first_lane(px[p]), first_lane(py[p]));
        if (lane == 0) s_box[wave * PPT + p] = b;
      }
      __syncthreads();
    }
    for (int i = threadIdx.x; i < cnt; i += nthreads) {
      const uint32_t rec = a.ids[bs + i];
      const float4 ra = a.splats[(size_t)rec * 3 + 0];
      const float4 rb = a.splats[(size_t)rec * 3 + 1];
      s_e[i] = a.pair_index[bs + i];
      s_a[i] = staged_a(ra);
      s_b[i] = staged_b(rb);
      s_c[i] = a.splats[(size_t)rec * 3 + 2];
      if (CULL) s_mask[i] = (uint16_t)footprint_mask(ra, rb, nwaves * PPT, s_box);
    }
    const int nchunks = (cnt + kWave - 1) / kWave;
#pragma unroll 1
    for (int i = threadIdx.x; i < (int)(part_bytes(batch, nwaves) / 16); i += nthreads)
      ((float4*)s_part)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    for (int c = nchunks - 1; c >= 0; --c) {
      uint64_t mp[PPT];
      uint64_t m = chunk_bits<PPT, CULL>(s_mask, c, cnt, wave, lane, mp);
      if (m == 0) {
        if (lane == 0) s_hit[c][wave] = 0;
        continue;
      }
      uint64_t hit = 0;
      // one staged record's per-pixel partials x (u v A B C o' r g b) over the
      // lane's pixels; returns the lanes that composite it
      auto partials = [&](int j, const float4& ra, const float4& rb, const float4& rc, float (&x)[GS_GRAD_FLOATS]) {
        const int jr = (int)(bs - tc.start) + j;  // index within the tile's list
        const float hb = 0.5f * ra.w;             // staged b / 2
#pragma unroll
        for (int k = 0; k < GS_GRAD_FLOATS; ++k) x[k] = 0.0f;
        uint64_t any = 0;
#pragma unroll
        for (int p = 0; p < PPT; ++p) {
          if (PPT > 1 && !((mp[p] >> (j - c * kWave)) & 1ull)) continue;  // wave-uniform: the block is not reached
          Eval e;
          eval_splat_all(px[p], py[p], ra.x, ra.y, ra.z, ra.w, rb.x, rb.y, &e);
          const uint64_t use = lanes_inside(e, rb.z) & __ballot(jr < lc[p]) & __ballot(!(e.alpha < kAlphaMin));
          any |= use;
          // lanes that do not composite this splat are left out through the exec
          // mask, or with one block add exact zeros (fewer waves' work to hide
          // a branch behind)
          const bool in = lane_in(use);
          if (PPT == 1 || in) {
            const float inv = __builtin_amdgcn_rcpf(1.0f - e.alpha);
            T[p] = PPT > 1 || in ? T[p] * inv : T[p];  // transmittance in front of this splat
            const float wgt = PPT > 1 || in ? e.alpha * T[p] : 0.0f;
            x[6] += wgt * g0[p];
            x[7] += wgt * g1[p];
            x[8] += wgt * g2[p];
            const float cd = rc.x * g0[p] + rc.y * g1[p] + rc.z * g2[p];
            const float dLda = (PPT > 1 || in) && !(e.raw > kAlphaMax) ? T[p] * cd - RdL[p] * inv : 0.0f;
            RdL[p] += cd * wgt;
            x[5] += e.G * dLda;
            // m = alpha dL/dalpha = -2 dL/dq; the constant factors are applied once,
            // to the sums.  The conic of the position gradient is not: along a
            // needle a dx and b/2 dy nearly cancel in every pixel, and sums of m dx
            // and m dy, rounded before they meet the conic, leave an error of the
            // sums' size (half of the rows of 0.55 x 10 and 0.55 x 30 pixel needles
            // off by 1.9 to 3.1 units of 2^-24 of their products, here by 0.3 to
            // 0.5; no walk is slower for it).  The products are the evaluation's.
            const float m = e.alpha * dLda;
            const float mdx = m * e.dx, mdy = m * e.dy;
            x[0] += m * __builtin_fmaf(hb, e.dy, e.adx);
            x[1] += m * __builtin_fmaf(hb, e.dx, e.cdy);
            x[2] += mdx * e.dx;
            x[3] += mdx * e.dy;
            x[4] += mdy * e.dy;
          }
        }
        return any;
      };
      float* my_part = s_part + wave * batch * GS_GRAD_FLOATS + my_e;
      // two records at a time, back to front: two independent chains up to the
      // transmittance, and one reduction (one record at a time, the next one's
      // reads ahead of it, took 43 us where this takes 40 at 2K Gaussians, 138 -> 131 at
      // 200K, 407 -> 394 for eight views of 1M, 397 -> 387 at two pixels a thread,
      // 2520 -> 2493 at four for 6M; reading the next two ahead costs as much again
      // in register copies)
      while (m != 0) {
        const int k0 = 63 - __builtin_clzll(m);
        m &= ~(1ull << k0);
        const bool two = m != 0;  // else the second set repeats the first and is left out
        const int k1 = two ? 63 - __builtin_clzll(m) : k0;
        m &= ~(1ull << k1);
        const int j0 = c * kWave + k0, j1 = c * kWave + k1;
        const float4 a0 = s_a[j0], b0 = s_b[j0], c0 = s_c[j0];
        const float4 a1 = s_a[j1], bb1 = s_b[j1], c1 = s_c[j1];
        __builtin_amdgcn_sched_barrier(0);  // all in flight together
        float x[GS_GRAD_FLOATS], y[GS_GRAD_FLOATS];
        const uint64_t any0 = partials(j0, a0, b0, c0, x);
        // a repeated record is left out by its distance
        const uint64_t any1 = partials(j1, two ? a1 : make_float4(__builtin_nanf(""), a1.y, a1.z, a1.w), bb1, c1, y);
        if ((any0 | any1) != 0) {  // wave-uniform: the whole wave takes part
          if (any0 != 0) hit |= 1ull << k0;
          if (any1 != 0) hit |= 1ull << k1;
          const float v = reduce_scatter9x2(x, y, b1, b2, b3);
          const int row = lane < kWave / 2 ? j0 * GS_GRAD_FLOATS : j1 * GS_GRAD_FLOATS;
          const uint64_t rows = (any0 != 0 ? 0xffffffffull : 0ull) | (any1 != 0 ? 0xffffffffull << 32 : 0ull);
          if (writer && lane_in(rows)) my_part[row] = v * escale;
        }
      }
      if (lane == 0) s_hit[c][wave] = hit;
    }
    __syncthreads();
    // the entries with rows, in order
    int rows = 0;
#pragma unroll 1
    for (int c = 0; c < nchunks; ++c) {
      uint64_t h = 0;
#pragma unroll 1
      for (int w = 0; w < nwaves; ++w) h |= s_hit[c][w];
      if (a.zero_rows) h = cnt - c * kWave < kWave ? (1ull << (cnt - c * kWave)) - 1ull : ~0ull;
      if (wave == c % nwaves && ((h >> lane) & 1ull))
        L.row[rows + __popcll(h & ((1ull << lane) - 1ull))] = (uint16_t)(c * kWave + lane);
      rows += __popcll(h);
    }
    __syncthreads();
    // fixed-order sum over the waves, one store per (pair, attribute)
    for (int i = threadIdx.x; i < rows * GS_GRAD_FLOATS; i += nthreads) {
      const int r = i / GS_GRAD_FLOATS, k = i - r * GS_GRAD_FLOATS, j = L.row[r];
      float v = s_part[j * GS_GRAD_FLOATS + k];
      for (int w = 1; w < nwaves; ++w) v += s_part[(w * batch + j) * GS_GRAD_FLOATS + k];
      grad_pair[(size_t)s_e[j] * GS_GRAD_FLOATS + k] = v;
      if (k == 0) a.pair_live[s_e[j]] = 1;
    }
    __syncthreads();
    be = bs;
  }
}

// Takes 67 registers at 1 pixel a thread (seven waves per SIMD; its LDS allows
// six); held to 80 and 96 at 2 and 4 (six and five; at 4 it takes more without,
// and 2760 us for 2493; held, it spills one).
template <int PPT>
constexpr int bwd_waves() { return PPT <= 2 ? 6 : 5; }
template <int PPT, bool CULL>
__global__ __launch_bounds__(256, bwd_waves<PPT>()) void render_bwd_kernel(RenderArgs a, ViewTable vt,
                                                         const float* __restrict__ T_final,
                                                         const int32_t* __restrict__ last_in,
                                                         const float* __restrict__ dL_dimage,
                                                         float* __restrict__ grad_pair) {
  extern __shared__ __align__(16) unsigned char smem[];
  LossIn loss;
  loss.dL_dimage = dL_dimage;
  loss.image = loss.target = nullptr;
  loss.dL_out = nullptr;
  bwd_item<PPT, CULL, false>(a, vt, T_final, last_in, loss, grad_pair, (int64_t)blockIdx.x, smem);
}

// Backward work list of the one-launch walks.  Each tile contributes its first
// chunk and one item per boundary (start + k 2^log2_chunk, k >= 1, whether or
// not the forward walk reaches it: a chunk past the walk then finds nothing to
// do).  Tiles are grouped by the bit length of their list length and the groups
// laid out lightest first: a tile's backward items are then taken about when its
// forward walk ends, and the deepest lists' items, whose forward walks end last,
// come last (an item taken before its tile's forward walk has ended holds its
// workgroup slot while it waits).  An entry is a render_bwd_kernel item number
// with the schedule off: a boundary chunk is its slot, tile t's first chunk
// nslots + t.  The count pass also records each boundary's owner.
// hist: [0, 64) items per group, [64, 128) write positions, [128] the total.
__device__ __forceinline__ int list_group(uint32_t len) { return len ? 32 - __clz(len) : 0; }

__device__ __forceinline__ uint32_t list_items(uint32_t len, int lg) {
  return (uint64_t)len > (1ull << lg) ? (uint32_t)(((uint64_t)len - 1) >> lg) + 1u : 1u;
}

__device__ __forceinline__ uint32_t list_len(const RenderArgs& a, int64_t t) {
  return *a.status == 0 ? a.ranges[2 * t + 1] - a.ranges[2 * t] : 0u;
}

__global__ __launch_bounds__(256) void list_count_kernel(RenderArgs a, int64_t tiles, uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[64];
  if (threadIdx.x < 64) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < tiles) {
    const uint32_t len = list_len(a, t);
    const int lg = a.log2_chunk;
    const uint64_t start = a.ranges[2 * t];
    for (uint64_t q = start + (1ull << lg); q < start + len; q += 1ull << lg) a.slot_owner[q >> lg] = (uint32_t)t;
    atomicAdd(&h[list_group(len)], list_items(len, lg));
  }
  __syncthreads();
  if (threadIdx.x < 64 && h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

__global__ void list_scan_kernel(uint32_t* __restrict__ hist) {
  if (threadIdx.x != 0) return;
  uint32_t run = 0;
  for (int g = 0; g < 64; ++g) {
    hist[64 + g] = run;
    run += hist[g];
  }
  hist[128] = run;
}

__global__ __launch_bounds__(256) void list_scatter_kernel(RenderArgs a, int64_t tiles, uint32_t* __restrict__ hist,
                                                           uint32_t* __restrict__ list) {
  // offsets within the block per group (LDS), one global reservation per group and block
  __shared__ uint32_t h[64], base[64];
  if (threadIdx.x < 64) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lg = a.log2_chunk;
  int g = 0;
  uint32_t len = 0, n = 0, off = 0;
  if (t < tiles) {
    len = list_len(a, t);
    g = list_group(len);
    n = list_items(len, lg);
    off = atomicAdd(&h[g], n);
  }
  __syncthreads();
  if (threadIdx.x < 64 && h[threadIdx.x]) base[threadIdx.x] = atomicAdd(&hist[64 + threadIdx.x], h[threadIdx.x]);
  __syncthreads();
  if (t >= tiles) return;
  uint32_t* out = list + base[g] + off;
  out[0] = (uint32_t)(a.nslots + t);
  const uint64_t start = a.ranges[2 * t];
  for (uint32_t k = 1; k < n; ++k) out[k] = (uint32_t)((start + ((uint64_t)k << lg)) >> lg);
}

// Polls (at most kWaitPolls times, sleeping about 2000 cycles between polls)
// until the flag is set; its value, or 0 if it never was (after about a second).
constexpr int kWaitPolls = 1 << 20;
__device__ __forceinline__ uint32_t wait_flag(const uint32_t* flag) {
  for (int i = 0; i < kWaitPolls; ++i) {
    const uint32_t v = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (v != 0u) return v;
    __builtin_amdgcn_s_sleep(32);
  }
  return 0u;
}

// Forward and backward walks in one launch, for the mean-squared-error loss
// (the loss gradient of a pixel needs only that pixel).  Each workgroup takes
// the next work item from a ticket: first every tile's forward walk in the
// heaviest-first schedule, then the backward work list (lightest lists first,
// see list_count_kernel).  A forward item sets its tile's flag once the image,
// T_final, last_contrib and chunk states of the tile are written; a backward
// item waits for its tile's flag, which holds 1 + the tile's largest
// last_contrib (a boundary chunk past it then leaves at once).  The flags it
// waits for belong to items taken earlier, which wait for nothing, so every
// wait ends (a wait that outlives its poll limit gives up and makes the item's
// gradients NaN instead of blocking).
// The backward items of finished tiles run while the deepest tiles' forward
// walks are still going.  sync: [total_tiles] flags, the ticket, all zero at
// launch, then the list's counts (kListHist words) and the list.
// At one pixel a thread the kernel is held to 80 registers (six waves per SIMD,
// as many as the backward's LDS allows), though its forward then spills 12.  Held
// to 96 (five waves, none spilled) it is as fast: eight views of 1M Gaussians in
// 16 x 16 tiles 1.234 ms for 1.230 at 512-entry backward chunks and 1.571 for 1.577
// at 256, 200K Gaussians 0.289 for 0.292 and 0.280 for 0.273, in 16 x 8 tiles 0.361
// for 0.372; not held (99) 1.288, 1.597, 0.306 and 0.288.
template <int PPT, bool CULL>
__global__ __launch_bounds__(256, PPT == 1 ? 6 : 1) void render_fused_kernel(RenderArgs a, ViewTable vt,
                                                                             float* __restrict__ image,
                                                                             float* __restrict__ T_final,
                                                                             int32_t* __restrict__ last, LossIn loss,
                                                                             float* __restrict__ grad_pair,
                                                                             uint32_t* __restrict__ sync) {
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ uint32_t s_ticket;
  __shared__ uint32_t s_flag;
  __shared__ int s_wmax[4];
  const int64_t ntiles = vt.total_tiles;
  if (threadIdx.x == 0) s_ticket = atomicAdd(sync + ntiles, 1u);
  __syncthreads();
  const int64_t q = s_ticket;
  if (q < ntiles) {
    // forward walks issue ahead of the backward waves that share their SIMD:
    // the deepest lists' forward walks are the launch's critical path
    __builtin_amdgcn_s_setprio(3);
    int my_max = fwd_item<PPT, CULL, kFull, true>(
        a, vt, image, T_final, last, q, (float4(*)[3][kWave])smem);
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) my_max = max(my_max, __shfl_xor(my_max, o, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0) s_wmax[threadIdx.x / kWave] = my_max;
    // every thread's coherent stores of image, T_final, last_contrib and
    // states have been acknowledged before the flag is set
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (threadIdx.x == 0) {
      int m = 0;
      for (int w = 0; w < (int)blockDim.x / kWave; ++w) m = max(m, s_wmax[w]);
      const int gtile = a.order ? (int)a.order[q] : (int)q;
      // the flag: 1 + the largest last_contrib of the tile
      __hip_atomic_store(sync + gtile, (uint32_t)m + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return;
  }
  const uint32_t* hist = sync + ntiles + 1;
  const int64_t qb = q - ntiles;
  if (qb >= (int64_t)hist[128]) return;  // past the list (the grid is sized for the most items)
  const int64_t item = hist[kListHist + qb];
  RenderArgs ab = a;
  ab.order = nullptr;  // first chunks are numbered by tile
  if (threadIdx.x == 0) {
    int gtile = -1;
    if (item < a.nslots) {
      const uint32_t owner = a.slot_owner[item];
      if (owner < (uint32_t)ntiles) gtile = (int)owner;
    } else {
      gtile = (int)(item - a.nslots);
    }
    s_flag = gtile < 0 ? 1u : wait_flag(sync + gtile);
  }
  __syncthreads();  // the tile's values are then read with coherent loads
  // a flag never seen set: the item's loss gradient, hence its gradients, are NaN
  const uint32_t f = s_flag;
  bwd_item<PPT, CULL, true>(ab, vt, T_final, last, loss, grad_pair, item, smem, f != 0u, f != 0u ? (int)(f - 1u) : -1);
}

static int tile_threads(const RenderArgs& a) { return (1 << (a.log2_tw + a.log2_th)) / a.ppt; }

// Work items [item_base, item_base + items) of one walk launch.
template <int PPT, int MODE>
static void walk(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final, int32_t* last,
                 int64_t item_base, int64_t items, hipStream_t s) {
  if (items <= 0) return;
  const int nt = tile_threads(a);
  const dim3 grid((unsigned)items), block((unsigned)nt);
  if (a.cull)
    hipLaunchKernelGGL((render_fwd_kernel<PPT, true, MODE>), grid, block, 0, s, a, vt, image, T_final, last,
                       item_base);
  else
    hipLaunchKernelGGL((render_fwd_kernel<PPT, false, MODE>), grid, block, 0, s, a, vt, image, T_final, last,
                       item_base);
}

template <int PPT>
static void fwd_ppt(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final, int32_t* last,
                    hipStream_t s) {
  if (a.nfslots > 0)
    hipLaunchKernelGGL(fwd_mark_kernel, dim3((unsigned)((vt.total_tiles + 255) / 256)), dim3(256), 0, s, a,
                       vt.total_tiles);
  walk<PPT, kFull>(a, vt, image, T_final, last, a.nfslots, vt.total_tiles, s);  // every tile's first chunk
  if (a.nfslots > 0) {
    walk<PPT, kTPass>(a, vt, nullptr, nullptr, nullptr, 0, a.nfslots, s);  // products of chunks 1 .. m-2
    walk<PPT, kFull>(a, vt, image, T_final, last, 0, a.nfslots, s);       // chunks 1 .. m-1
    hipLaunchKernelGGL((fwd_combine_kernel<PPT>), dim3((unsigned)vt.total_tiles), dim3((unsigned)tile_threads(a)), 0,
                       s, a, vt, image, T_final, last);
  }
}

template <int PPT>
static void count_ppt(const RenderArgs& a, const ViewTable& vt, hipStream_t s) {
  walk<PPT, kCount>(a, vt, nullptr, nullptr, nullptr, 0, vt.total_tiles, s);
}

template <int PPT>
static void bwd_ppt(const RenderArgs& a, const ViewTable& vt, const float* T_final, const int32_t* last,
                    const float* dL, float* grad_pair, hipStream_t s) {
  const int nt = tile_threads(a);
  // chunk items first, then one item per tile
  const dim3 grid((unsigned)(a.nslots + vt.total_tiles)), block((unsigned)nt);
  const size_t sh = lds_bytes(bwd_batch(a.batch, nt / kWave), nt / kWave, true);
  if (a.cull)
    hipLaunchKernelGGL((render_bwd_kernel<PPT, true>), grid, block, sh, s, a, vt, T_final, last, dL, grad_pair);
  else
    hipLaunchKernelGGL((render_bwd_kernel<PPT, false>), grid, block, sh, s, a, vt, T_final, last, dL, grad_pair);
}

hipError_t launch_render_fwd(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final,
                             int32_t* last_contrib, hipStream_t s) {
  if (vt.total_tiles == 0) return hipSuccess;
  hipError_t e = launch_fill_u32(a.slot_owner, a.nslots, 0xffffffffu, s);  // no boundary recorded yet
  if (e != hipSuccess) return e;
  if (a.nfslots > 0 && (e = launch_fill_u32(a.fslot_owner, a.nfslots, 0xffffffffu, s)) != hipSuccess) return e;
  switch (a.ppt) {
    case 1: fwd_ppt<1>(a, vt, image, T_final, last_contrib, s); break;
    case 2: fwd_ppt<2>(a, vt, image, T_final, last_contrib, s); break;
    default: fwd_ppt<4>(a, vt, image, T_final, last_contrib, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_count_hits(const RenderArgs& a, const ViewTable& vt, hipStream_t s) {
  if (vt.total_tiles == 0) return hipSuccess;
  switch (a.ppt) {
    case 1: count_ppt<1>(a, vt, s); break;
    case 2: count_ppt<2>(a, vt, s); break;
    default: count_ppt<4>(a, vt, s); break;
  }
  return hipGetLastError();
}

template <int PPT>
static void fused_ppt(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final, int32_t* last,
                      const LossIn& loss, float* grad_pair, uint32_t* sync, hipStream_t s) {
  const int nt = tile_threads(a);
  const size_t bwd_sh = lds_bytes(bwd_batch(a.batch, nt / kWave), nt / kWave, true);
  const size_t fwd_sh = sizeof(float4) * 4 * 3 * kWave;
  const size_t sh = bwd_sh > fwd_sh ? bwd_sh : fwd_sh;
  // forward items, then at most one backward item per tile and one per boundary slot
  const dim3 grid((unsigned)(2 * vt.total_tiles + a.nslots)), block((unsigned)nt);
  if (a.cull)
    hipLaunchKernelGGL((render_fused_kernel<PPT, true>), grid, block, sh, s, a, vt, image, T_final, last, loss,
                       grad_pair, sync);
  else
    hipLaunchKernelGGL((render_fused_kernel<PPT, false>), grid, block, sh, s, a, vt, image, T_final, last, loss,
                       grad_pair, sync);
}

hipError_t launch_render_fused(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final,
                               int32_t* last_contrib, const float* target, const float* scale, float* dL_out,
                               float* grad_pair, uint32_t* sync, hipStream_t s) {
  if (vt.total_tiles == 0) return hipSuccess;
  if (a.nfslots != 0) return hipErrorInvalidValue;  // forward chunking runs as separate launches
  LossIn loss;
  loss.dL_dimage = nullptr;
  loss.image = image;
  loss.target = target;
  loss.dL_out = dL_out;
  for (int v = 0; v < GS_MAX_VIEWS; ++v) loss.scale[v] = v < vt.nviews ? scale[v] : 0.0f;
  hipError_t e = launch_fill_u32(a.slot_owner, a.nslots, 0xffffffffu, s);
  if (e == hipSuccess) e = launch_fill_u32(sync, vt.total_tiles + 1 + 64, 0u, s);  // flags, ticket, list counts
  if (e != hipSuccess) return e;
  uint32_t* hist = sync + vt.total_tiles + 1;
  const dim3 tgrid((unsigned)((vt.total_tiles + 255) / 256));
  hipLaunchKernelGGL(list_count_kernel, tgrid, dim3(256), 0, s, a, (int64_t)vt.total_tiles, hist);
  hipLaunchKernelGGL(list_scan_kernel, dim3(1), dim3(64), 0, s, hist);
  hipLaunchKernelGGL(list_scatter_kernel, tgrid, dim3(256), 0, s, a, (int64_t)vt.total_tiles, hist,
                     hist + kListHist);
  switch (a.ppt) {
    case 1: fused_ppt<1>(a, vt, image, T_final, last_contrib, loss, grad_pair, sync, s); break;
    case 2: fused_ppt<2>(a, vt, image, T_final, last_contrib, loss, grad_pair, sync, s); break;
    default: fused_ppt<4>(a, vt, image, T_final, last_contrib, loss, grad_pair, sync, s); break;
  }
  return hipGetLastError();
}

hipError_t launch_render_bwd(const RenderArgs& a, const ViewTable& vt, const float* T_final,
                             const int32_t* last_contrib, const float* dL_dimage, float* grad_pair, hipStream_t s) {
  if (vt.total_tiles == 0) return hipSuccess;
  switch (a.ppt) {
    case 1: bwd_ppt<1>(a, vt, T_final, last_contrib, dL_dimage, grad_pair, s); break;
    case 2: bwd_ppt<2>(a, vt, T_final, last_contrib, dL_dimage, grad_pair, s); break;
    default: bwd_ppt<4>(a, vt, T_final, last_contrib, dL_dimage, grad_pair, s); break;
  }
  return hipGetLastError();
}

}  // namespace gs
