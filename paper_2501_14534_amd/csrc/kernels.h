// Kernel argument structs and launch wrappers of libgs (host + device).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gs_common.h"

namespace gs {

struct ProjectArgs {
  const float* means;
  const float* log_scales;
  const float* quats;
  const float* opacity_logits;
  const float* sh_dc;
  const float* sh_rest;
  const float* mask_logits;
  const float* sh_mask_logits;
  int64_t n;
  float mask_thr;     // logit(mask_eps), rounded down to float
  float sh_mask_thr;  // logit(sh_mask_eps), rounded down to float
  float near_plane;
  float inv_tw, inv_th;
  float4* splats;
  uint32_t* tiles_touched;
};

struct RenderArgs {
  const float4* splats;
  const uint32_t* ids;
  const uint32_t* pair_index;
  uint8_t* pair_live;     // backward: [capacity] 1 where the pair's gradient row was written
  const uint32_t* ranges;
  const uint32_t* order;  // tile schedule (NULL: tile-id order)
  const int32_t* status;
  int32_t log2_tw, log2_th;
  int32_t log2_sw, log2_sh;  // sub-tile (one per wave) width and height
  int32_t log2_sx;           // sub-tiles along x
  int32_t log2_bw, log2_bx;  // 64-pixel blocks of a sub-tile (one per pixel of a thread): width, blocks along x
  int32_t batch;
  int32_t ppt;
  int32_t cull;
  int32_t zero_rows;  // backward: also write the rows (zeros) of the walked pairs that no pixel composites
  float bg[3];
  // per-chunk pixel states written by the forward, read by the backward:
  // boundary position q = start + k * 2^log2_chunk (k >= 1) of a tile's list
  // owns slot q >> log2_chunk; slot_owner[slot] = global tile, state[slot][pixel]
  // = (T, colour composited after q)
  int32_t log2_chunk;
  int64_t nslots;
  uint32_t* slot_owner;
  float4* state;
  // hit counting (Eq. 4): per-Gaussian counters, n Gaussians per view
  uint32_t* hits;
  int64_t n;
  // forward chunking: lists longer than 2^log2_fchunk entries (31: off) are
  // walked in chunks by separate workgroups.  Forward boundary q = start + kF
  // (k >= 1) owns slot q >> log2_fchunk: fslot_owner[slot] = global tile;
  // fprod[slot][pixel] = product of (1 - alpha) over the chunk ending at q;
  // fres/flast[slot] = (colour, final T) / last index of the chunk ending at
  // q, and at [nfslots + slot] those of a list's last chunk starting at q;
  // fsuf[slot] = colour composited from q on (read by the backward).
  int32_t log2_fchunk;
  int64_t nfslots;
  uint32_t* fslot_owner;
  float* fprod;
  float4* fres;
  int32_t* flast;
  float4* fsuf;
};

struct BinOut {
  uint64_t* keys;
  uint32_t* ids;
  uint32_t* pair_index;
  uint32_t* offsets;
  uint32_t* ranges;
  uint32_t* order;
  uint32_t* count;
  int32_t* status;
};

struct ProjectBwdArgs {
  ProjectArgs p;                   // forward inputs (outputs unused)
  const float* grad_pair;          // [K][9], emission order
  const uint32_t* tiles_touched;   // [V*n]
  const uint32_t* offsets;         // [V*n] first emission position of each record
  const uint8_t* pair_live;        // [K] 1 where the walk wrote the pair's row (others count as zero)
  const int32_t* status;
  float* rec;                      // [V][nwaves][64][12] packed record gradients of 64 Gaussians
  uint64_t* rec_mask;              // [V][nwaves] the lanes that are packed
  int64_t nwaves;                  // n / 64, rounded up
  float* g_means;
  float* g_log_scales;
  float* g_quats;
  float* g_opacity_logits;
  float* g_sh_dc;
  float* g_sh_rest;
  float* g_mask_logits;
  float* g_sh_mask_logits;
  float* g_mean2d;
  int32_t assign;                  // 1: write the parameter gradients (zeros where none), 0: add them
};

// Views of an image call (loss: 116 x 16 tiles; target blur: blur_tile_w(r) x 16): per
// view its size, tile grid, tile width, pixel offset (views concatenated, each
// [3][H][W]) and first workgroup; the loss window's taps.  The tiles have the width
// above, except where the last one of a row would keep at most kFewColumns: they
// leave the row passes at most 8 lanes of a wave, where the same arithmetic takes
// 1.4 times as long.  Such rows are cut into about equal tiles (the loss of one 128
// x 128 view 20.5 us, with two tiles of 64 columns 15.7).
constexpr int kFewColumns = 16;
constexpr int kLossTileW = 116, kLossTileH = 16;
constexpr int kBlurTileH = 16;
__host__ __device__ constexpr int blur_tile_w(int r) { return 128 - (2 * r + 3) / 4 * 4; }
struct LossView {
  int32_t W, H, TX, TY, tw;
  int64_t pix_off;
  int32_t block_off;
};
struct LossViews {
  LossView v[GS_MAX_VIEWS];
  int32_t nviews;
  int32_t total_blocks;
  float g[11];  // normalised Gaussian taps of the 11 x 11 window's 1-D factor
};

// Workgroups of an image call, 256 threads each.  A launch holds fewer than 2^32
// threads, so past 2^23 workgroups (a 1 x 4.5e7 image's tiles) it takes several:
// launch(first workgroup, their number).  (Rows of workgroups in one launch need a
// check at the last one's end, a load that each workgroup waits for: 44.2 us for the
// loss of a 1264 x 832 view, 43.6 without.)
template <typename F>
inline void image_launches(int64_t nb, F launch) {
  constexpr int64_t kMost = 1 << 23;
  for (int64_t first = 0; first < nb; first += kMost)
    launch((int)first, dim3((unsigned)(nb - first < kMost ? nb - first : kMost)));
}

// Workgroup b of an image call: its view, colour plane and tile.
struct LossTile {
  int view, plane, tx, ty;
};

__device__ __forceinline__ LossTile loss_tile(const LossViews& lv, int b) {
  LossTile t;
  int v = 0;
  while (v + 1 < lv.nviews && b >= lv.v[v + 1].block_off) ++v;
  const LossView& q = lv.v[v];
  const int lb = b - q.block_off;
  const int per_plane = q.TX * q.TY;
  t.view = v;
  t.plane = lb / per_plane;
  const int r = lb - t.plane * per_plane;
  t.ty = r / q.TX;
  t.tx = r - t.ty * q.TX;
  return t;
}

// Target blur: the views' tiles, radius r = (k - 1) / 2 and the k taps.
constexpr int kMaxBlurRadius = 15;
struct BlurArgs {
  LossViews views;
  int32_t r;
  float g[2 * kMaxBlurRadius + 1];
};

// Mean squared error gradient: per view the end of its elements and the scale.
struct L2Args {
  int64_t end[GS_MAX_VIEWS];  // exclusive end of view v's 3 H W elements
  float scale[GS_MAX_VIEWS];  // 2 / (3 H W mean_views)
  int32_t nviews;
};
hipError_t launch_l2_grad(const float* image, const float* target, float* dL, const L2Args& a, hipStream_t s);
// Forward and backward walks in one launch with the mean-squared-error gradient
// dL = scale[v] (image - target) computed inline (render.hip).  Needs forward
// chunking off; pair_live cleared by the caller; sync: fused_sync_words u32
// (tile flags, the ticket, kListHist counts of the backward work list, the list).
constexpr int kListHist = 129;
inline int64_t fused_sync_words(int64_t total_tiles, int64_t nslots) {
  return total_tiles + 1 + kListHist + total_tiles + nslots;
}
hipError_t launch_render_fused(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final,
                               int32_t* last_contrib, const float* target, const float* scale, float* dL_out,
                               float* grad_pair, uint32_t* sync, hipStream_t s);

// Target resize: per view the input and output sizes and pixel offsets, the
// output values of a row that a workgroup takes (their boxes fit kResizeCols
// input columns where one does), the stretches of a row and the first of the
// view's 3 H' nseg stretches.
constexpr int kResizeCols = 1024;
struct ResizeView {
  int32_t W, H, Wo, Ho;
  int64_t in_off, out_off;
  float inv_area;  // 1 / (W H)
  int32_t seg, nseg;
  int64_t item_off;
};
struct ResizeArgs {
  ResizeView v[GS_MAX_VIEWS];
  int32_t nviews;
  int32_t by_box;     // one thread per output value instead
  int64_t items;
  int64_t total_out;  // 3 * sum of W' H'
};

hipError_t launch_blur(const float* in, float* out, const BlurArgs& b, hipStream_t s);
hipError_t launch_resize(const float* in, float* out, const ResizeArgs& a, hipStream_t s);

hipError_t launch_loss(const LossViews& lv, const float* image, const float* target, float lambda, float* loss,
                       float* dL, float* dmap, float* bsum, double* per_view, hipStream_t s);

hipError_t launch_mask_loss(const float* m, const float* msh, int64_t n, int deg, float lam_m, float lam_sh,
                            float* gm, float* gsh, float* loss, float* bsum, hipStream_t s);

// Radix-select state of the volume quantile (significance score).
struct SelectState {
  uint32_t prefix[4];  // before pass p: key bits chosen so far
  uint32_t rank[4];    // and the rank still wanted among the keys matching them
  uint32_t hist[4][256];
};

hipError_t launch_significance(const float* log_scales, const float* opacity_logits, const float* mask_logits,
                               float mask_thr, const uint32_t* hits, int64_t n, uint32_t rank, SelectState* st,
                               float* score, hipStream_t s);

// Workspace carve-up of gs_bin_sort / gs_render_bwd.
struct SortPlan {
  int64_t nrec;             // V * n
  uint64_t capacity;        // pair capacity
  int64_t rec_blocks;       // records / 4096 (count and compaction)
  int64_t scan_blocks;      // records / 1024 (emission of the visible records)
  int64_t rec_sort_blocks;  // records / 4096 (depth sort of the visible records)
  int64_t sort_blocks;      // capacity / 4096 (tile sort of the pairs)
  int tile_bits;            // ceil(log2 #tiles), sorted in passes of 8
};

hipError_t launch_project(const ProjectArgs& a, const ViewTable& vt, int deg, hipStream_t s);

hipError_t launch_bin_sort(const SortPlan& plan, const float4* splats, const uint32_t* tiles_touched, int64_t n,
                           const ViewTable& vt, float inv_tw, float inv_th, const BinOut& out, uint64_t capacity,
                           void* ws, hipStream_t s);

hipError_t launch_render_fwd(const RenderArgs& a, const ViewTable& vt, float* image, float* T_final,
                             int32_t* last_contrib, hipStream_t s);

hipError_t launch_count_hits(const RenderArgs& a, const ViewTable& vt, hipStream_t s);

hipError_t launch_render_bwd(const RenderArgs& a, const ViewTable& vt, const float* T_final,
                             const int32_t* last_contrib, const float* dL_dimage, float* grad_pair, hipStream_t s);

hipError_t launch_project_bwd(const ProjectBwdArgs& a, const ViewTable& vt, int deg, hipStream_t s);

hipError_t launch_fill_u32(uint32_t* p, int64_t count, uint32_t value, hipStream_t s);

size_t bin_sort_ws_bytes(const SortPlan& plan);

}  // namespace gs
