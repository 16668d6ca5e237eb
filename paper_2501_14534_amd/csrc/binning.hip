// Tile binning and (tile, depth) ordering of projected records, depth first.
//
// Up to the emission, on more than 12288 records:
//   1. count_reduce + scan_top: device-wide exclusive scans of tiles_touched
//      (the canonical emission offsets, K and the capacity status) and of
//      the visibility flags (tiles_touched > 0), 4096 records per block.
//   2. compact_visible: writes each record's canonical offset and packs each
//      visible record as (depth bits, compact index) plus a 16-byte emission
//      descriptor (first tile, rect width and height, canonical offset, id).
//   3. LSD radix sort of the visible records by their 32 depth bits (four
//      8-bit passes; stable, so equal depths keep record order).
//   4. gather_reduce gathers the descriptors into depth order once (the only
//      random access of the emission) and sums the pairs per block;
//      scan_top and emit_prefix: each depth-sorted record's first output position.
// On fewer, small_lists leaves the same words in one workgroup, its depth sort in
// LDS: there the launches are most of the time (measured at small_lists).
// Then, on any number:
//   5. emit_pairs: the records, now in depth order, emit one (tile, canonical
//      pair index, record id) per touched tile into a contiguous
//      depth-ordered range; each workgroup fills a fixed chunk of output
//      positions slot by slot (the owning records by a running maximum over the
//      chunk), so writes are coalesced and neither a big Gaussian nor a block
//      of them serialises the work.
//   6. LSD radix sort of the pairs by tile id only (ceil(log2 #tiles) bits,
//      two passes up to 65536 tiles), carrying pair index and record id.
//      Stability keeps depth order, and record order among equal depths,
//      inside every tile: the order of a sort by (tile << 32 | depth bits)
//      then record id.
//   7. tile_ranges: [start, end) of every tile and, if asked for, the 64-bit keys.
//   8. tile_order_*: the heaviest-first tile schedule.
// A pass moves 8 bytes per visible record (4 passes) and 12 per pair (2 passes),
// instead of 6 passes of 16 over the pairs.  Each: per-block digit histogram (the
// pairs' first is counted by the emission), per-digit scan across blocks (up to
// kScanBlocks of them summed by the scatter itself), stable scatter ranked with
// 64-lane ballots.  Every kernel reads its element count from device memory, so
// nothing waits for the host.
#include "gs_common.h"
#include "kernels.h"

namespace gs {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 4;
constexpr int kScanTile = kScanThreads * kScanItems;  // depth-sorted records per emission scan block
constexpr int kRecTile = 4 * kScanTile;               // records per scan block: four rounds of kScanTile
constexpr int kSortThreads = 512;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;  // keys per sort block
constexpr int kRadix = 256;
// Sort blocks up to which a scatter sums the histogram's rows itself instead of
// after a launch of their scan: 256 rows of at most 256 bytes a block.  A call on
// 21 thousand records (six blocks a depth pass, 43 a tile pass): 137 -> 112 us; 49
// and 407 blocks: four scans of 4 us less, each scatter 1.5 us more.
constexpr int64_t kScanBlocks = 64;

__device__ __forceinline__ uint32_t effective_count(const uint32_t* count, const int32_t* status) {
  return *status != 0 ? 0u : *count;
}

// Data block of workgroup p among the first `nact` workgroups: workgroups are
// dealt round-robin to the 8 XCDs, so p % 8 is p's XCD; the remap gives each
// XCD a contiguous stretch of data blocks.  Neighbouring blocks share the
// cache lines at the ends of their output runs (the scatter) and the lines
// of their histogram column (32 blocks per line), which are then completed in
// one L2 and written back whole.
__device__ __forceinline__ int64_t xcd_block(int64_t p, int64_t nact) {
  constexpr int kXcds = 8;
  const int64_t q = nact / kXcds;
  return p < q * kXcds ? (p % kXcds) * q + p / kXcds : p;
}

// Exclusive scan of one value per thread over a 256-thread block.
__device__ __forceinline__ uint32_t block_exclusive_scan_256(uint32_t x, uint32_t* total, uint32_t* s_wave) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t incl = x;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += y;
  }
  if (lane == kWave - 1) s_wave[wave] = incl;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kScanThreads / kWave; ++w) {
    const uint32_t c = s_wave[w];
    off += (w < wave) ? c : 0u;
    tot += c;
  }
  __syncthreads();
  *total = tot;
  return incl - x + off;
}

// Four consecutive words of an array that is only word-aligned.
struct __attribute__((packed, aligned(4))) Words4 {
  uint32_t w[4];
};

// The caller's four consecutive records of round k of its block (0 past the end).
__device__ __forceinline__ void load_counts(const uint32_t* __restrict__ tt, int64_t r0, int64_t nrec,
                                            uint32_t c[kScanItems]) {
  if (r0 + kScanItems <= nrec) {
    const Words4 q = *(const Words4*)(tt + r0);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) c[j] = q.w[j];
  } else {
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) c[j] = r0 + j < nrec ? tt[r0 + j] : 0u;
  }
}

// Per block of 4096 records: sum of tiles_touched (saturated to 32 bits, which
// no capacity holds) and number of visible records.
__global__ __launch_bounds__(kScanThreads) void count_reduce(const uint32_t* __restrict__ tt, int64_t nrec,
                                                             uint2* __restrict__ block_sums) {
  __shared__ unsigned long long s_pairs[kScanThreads / kWave];
  __shared__ uint32_t s_vis[kScanThreads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kRecTile + (int64_t)threadIdx.x * kScanItems;
  unsigned long long s = 0;
  uint32_t v = 0;
#pragma unroll
  for (int k = 0; k < kRecTile / kScanTile; ++k) {
    uint32_t c[kScanItems];
    load_counts(tt, base + k * kScanTile, nrec, c);
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      s += c[j];
      v += c[j] != 0u;
    }
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    s += __shfl_xor(s, o, kWave);
    v += __shfl_xor(v, o, kWave);
  }
  if ((threadIdx.x & (kWave - 1)) == 0) s_pairs[threadIdx.x / kWave] = s, s_vis[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kScanThreads / kWave; ++w) s += s_pairs[w], v += s_vis[w];
    block_sums[blockIdx.x] = make_uint2(s > 0xffffffffull ? 0xffffffffu : (uint32_t)s, v);
  }
}

// Single block: exclusive scans of nb block sums in place, .x with 64-bit
// accumulation (the total saturated to 32 bits; with a status word, status = 1
// when it exceeds capacity), .y too where total_y is given.
// With a count, only the blocks of 1024 that hold that many entries.
__global__ __launch_bounds__(1024) void scan_top(uint2* __restrict__ sums, int64_t nb, const uint32_t* count,
                                                 uint64_t capacity, uint32_t* total_x, uint32_t* total_y,
                                                 int32_t* status) {
  constexpr int kItems = 4;  // consecutive sums per thread: 4096 per step, one step up to 16M records
  __shared__ unsigned long long s_wave[16];
  __shared__ uint32_t s_wave_y[16];
  __shared__ unsigned long long s_carry;
  __shared__ uint32_t s_carry_y;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  if (threadIdx.x == 0) s_carry = 0, s_carry_y = 0;
  if (count) nb = min(nb, ((int64_t)*count + 1023) / 1024);
  __syncthreads();
  for (int64_t base = 0; base < nb; base += kItems * 1024) {
    const int64_t i0 = base + (int64_t)kItems * threadIdx.x;
    uint2 x[kItems];
    unsigned long long sum = 0;
    uint32_t sum_y = 0;
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      x[j] = i0 + j < nb ? sums[i0 + j] : make_uint2(0u, 0u);
      sum += x[j].x;
      sum_y += x[j].y;
    }
    unsigned long long incl = sum;
    uint32_t incl_y = sum_y;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const unsigned long long a = __shfl_up(incl, o, kWave);
      const uint32_t b = __shfl_up(incl_y, o, kWave);
      if (lane >= o) incl += a, incl_y += b;
    }
    if (lane == kWave - 1) s_wave[wave] = incl, s_wave_y[wave] = incl_y;
    __syncthreads();
    unsigned long long off = 0, tot = 0;
    uint32_t off_y = 0, tot_y = 0;
    for (int w = 0; w < 16; ++w) {
      const unsigned long long c = s_wave[w];
      const uint32_t cy = s_wave_y[w];
      off += (w < wave) ? c : 0ull;
      off_y += (w < wave) ? cy : 0u;
      tot += c;
      tot_y += cy;
    }
    const unsigned long long carry = s_carry;
    const uint32_t carry_y = s_carry_y;
    uint2 ex = make_uint2((uint32_t)(carry + off + incl - sum), carry_y + off_y + incl_y - sum_y);
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      if (i0 + j < nb) sums[i0 + j] = ex;
      ex.x += x[j].x;
      ex.y += x[j].y;
    }
    __syncthreads();
    if (threadIdx.x == 0) s_carry = carry + tot, s_carry_y = carry_y + tot_y;
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const unsigned long long K = s_carry;
    *total_x = K > 0xffffffffull ? 0xffffffffu : (uint32_t)K;
    if (total_y) *total_y = s_carry_y;
    if (status) *status = K > (unsigned long long)capacity ? 1 : 0;
  }
}

// Canonical emission offsets of every record (pairs of record r occupy
// [offsets[r], offsets[r] + tiles_touched[r]), records in index order), and
// the visible records packed in record order as (depth bits, compact index)
// with their emission descriptors; drec[r] = depth bits for the keys.  Bound by
// HBM traffic: two words per record, and the lines of the visible records'
// splats, whose other half is not needed.  A block takes its 4096 records in
// rounds of 1024, four slices of 256 consecutive ones a round, so loads and
// stores are coalesced; the slices' wave sums meet at one barrier a round.
// (Four consecutive records a thread, one 16-byte load and store, read the
// splats at four times the stride: 103 -> 155 us at 8M records, 4M visible.)
__global__ __launch_bounds__(kScanThreads) void compact_visible(const float4* __restrict__ splats,
                                                                const uint32_t* __restrict__ tt, int64_t nrec,
                                                                int64_t n, ViewTable vt, float inv_tw, float inv_th,
                                                                const uint2* __restrict__ block_offsets,
                                                                const int32_t* __restrict__ status,
                                                                uint32_t* __restrict__ offsets,
                                                                uint32_t* __restrict__ dkey,
                                                                uint32_t* __restrict__ dval, uint4* __restrict__ desc,
                                                                uint32_t* __restrict__ drec) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ uint2 s_wave[2][kScanItems * kWaves];  // per slice and wave; two buffers in turn: one barrier a round
  if (*status != 0) return;  // overflow: no lists this step
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint2 base = block_offsets[blockIdx.x];
  for (int k = 0; k < kRecTile / kScanTile; ++k) {
    const int64_t r0 = (int64_t)blockIdx.x * kRecTile + k * kScanTile + threadIdx.x;
    if (r0 - threadIdx.x >= nrec) break;  // uniform
    uint32_t c[kScanItems], ex[kScanItems], vx[kScanItems];
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) c[j] = r0 + j * kScanThreads < nrec ? tt[r0 + j * kScanThreads] : 0u;
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      const uint32_t incl = wave_inclusive_sum(c[j]);
      const uint64_t vis = __ballot(c[j] != 0u);
      ex[j] = incl - c[j];
      vx[j] = (uint32_t)__popcll(vis & ((1ull << lane) - 1ull));
      if (lane == kWave - 1) s_wave[k & 1][j * kWaves + wave] = make_uint2(incl, (uint32_t)__popcll(vis));
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        if (w == wave) ex[j] += base.x, vx[j] += base.y;
        const uint2 q = s_wave[k & 1][j * kWaves + w];
        base.x += q.x;
        base.y += q.y;
      }
    }
#pragma unroll
    for (int j = 0; j < kScanItems; ++j) {
      const int64_t r = r0 + j * kScanThreads;
      if (r < nrec) offsets[r] = ex[j];
      if (c[j] == 0u) continue;
      const float2 uv = *(const float2*)(splats + r * 3);            // u, v
      const float2 rd = *((const float2*)(splats + r * 3 + 1) + 1);  // radius, depth
      int v = 0;
      while (v + 1 < vt.nviews && r >= (int64_t)(v + 1) * n) ++v;
      const ViewArgs& va = vt.v[v];
      int x0, y0, x1, y1;
      tile_rect(uv.x, uv.y, rd.x, inv_tw, inv_th, va.TX, va.TY, &x0, &y0, &x1, &y1);
      const uint32_t dbits = __float_as_uint(rd.y);  // depth > near plane > 0: bits order as values
      dkey[vx[j]] = dbits;
      dval[vx[j]] = vx[j];
      desc[vx[j]] = make_uint4((uint32_t)(va.tile_off + y0 * va.TX + x0),
                               (uint32_t)(x1 - x0 + 1) | ((uint32_t)(y1 - y0 + 1) << 16), ex[j], (uint32_t)r);
      if (drec) drec[r] = dbits;
    }
  }
}

// Per block of 1024 depth-sorted records: their descriptors gathered into
// depth order, (first tile, rect width | the view's tile columns << 16, first
// canonical pair, record), their output positions within the block, and the
// block's number of pairs.  Bound by the gather: 16 bytes of a line a record.
__global__ __launch_bounds__(kScanThreads) void gather_reduce(const uint4* __restrict__ desc,
                                                              const uint32_t* __restrict__ dval,
                                                              const uint32_t* __restrict__ nvis,
                                                              const int32_t* __restrict__ status, ViewTable vt,
                                                              uint4* __restrict__ sdesc, uint32_t* __restrict__ epref,
                                                              uint2* __restrict__ block_sums) {
  constexpr int kWaves = kScanThreads / kWave;
  __shared__ uint32_t s_wave[kScanItems * kWaves];
  const uint32_t N = effective_count(nvis, status);
  const int64_t blk = (int64_t)blockIdx.x * kScanTile;
  if (blk >= N) return;  // uniform: past the sums that are read
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint4 d[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t m = blk + k * kScanThreads + threadIdx.x;
    d[k] = m < N ? desc[dval[m]] : make_uint4(0u, 0u, 0u, 0u);
  }
  uint32_t ex[kScanItems];
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const uint32_t c = (d[k].y & 0xffffu) * (d[k].y >> 16), incl = wave_inclusive_sum(c);
    ex[k] = incl - c;
    if (lane == kWave - 1) s_wave[k * kWaves + wave] = incl;
  }
  __syncthreads();
  uint32_t run = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w == wave) ex[k] += run;
      run += s_wave[k * kWaves + w];
    }
    const int64_t m = blk + k * kScanThreads + threadIdx.x;
    if (m < N) {
      int v = 0;  // view of the record's first tile
      while (v + 1 < vt.nviews && d[k].x >= (uint32_t)vt.v[v + 1].tile_off) ++v;
      sdesc[m] = make_uint4(d[k].x, (d[k].y & 0xffffu) | ((uint32_t)vt.v[v].TX << 16), d[k].z, d[k].w);
      epref[m] = ex[k];
    }
  }
  if (threadIdx.x == 0) block_sums[blockIdx.x] = make_uint2(run, 0u);
}

// Output positions per emission workgroup, 8 per thread: a block of the tile
// sort, whose first digit's histogram the emission counts as it goes.
constexpr int kEmitItems = 8;
constexpr int kEmitThreads = kSortTile / kEmitItems;
constexpr int kEmitChunk = kSortTile;

// Emission offsets in depth order: epref[m], the position within its block of
// 1024, becomes the first output position of depth-sorted record m, and
// chunk_first of every chunk of kEmitChunk output positions the record holding
// its first position.
__global__ __launch_bounds__(kScanThreads) void emit_prefix(const uint32_t* __restrict__ nvis,
                                                            const uint32_t* __restrict__ count,
                                                            const uint2* __restrict__ eblock_offsets,
                                                            const int32_t* __restrict__ status,
                                                            uint32_t* __restrict__ epref,
                                                            uint32_t* __restrict__ chunk_first) {
  const uint32_t N = effective_count(nvis, status);
  const int64_t blk = (int64_t)blockIdx.x * kScanTile;
  if (blk >= N) return;  // uniform
  const uint32_t off = eblock_offsets[blockIdx.x].x;
  const int64_t next_blk = blk + kScanTile;
  const uint32_t end = next_blk < N ? eblock_offsets[blockIdx.x + 1].x : *count;  // the block's last position + 1
  const int64_t m0 = blk + (int64_t)threadIdx.x * kScanItems;
  uint32_t ex[kScanItems + 1];
#pragma unroll
  for (int k = 0; k <= kScanItems; ++k)
    ex[k] = m0 + k < min((int64_t)N, next_blk) ? off + epref[m0 + k] : end;
  __syncthreads();  // every position has been read
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (m0 + k >= N) break;
    epref[m0 + k] = ex[k];
    // chunks whose first position lies in [ex[k], ex[k + 1])
    for (uint32_t q = (ex[k] + kEmitChunk - 1) / kEmitChunk; q * (uint64_t)kEmitChunk < (uint64_t)ex[k + 1]; ++q)
      chunk_first[q] = (uint32_t)(m0 + k);
  }
}

// Emission in depth order: sorted record m emits, at output positions
// [epref[m], epref[m] + w h), its tiles in row-major order of its tile
// rectangle: tile id, the pair's canonical index offsets[r] + j, and r.
// Workgroup c owns output positions [c C, (c + 1) C), C = kEmitChunk.  The
// records from the one holding its first position to the one holding the next
// chunk's (at most C + 1: every record has a pair) mark the slots where they
// start; a running maximum over the slots then gives each its record, whose
// descriptor consecutive threads read from one or two cache lines.  (A binary
// search of the record in LDS, ten dependent reads a slot over 30 KB of staged
// descriptors, took 68 us for 14.1M pairs and left the first histogram to a pass
// of 30 us; now 60 us with it.)  Work per workgroup is bounded by C
// slots however many pairs one record has (the nearest Gaussians cover
// thousands of tiles), and consecutive threads write consecutive positions.
// hist (the tile sort's, nblk columns): column c counts the chunk's tile ids by
// their low digit.
__global__ __launch_bounds__(kEmitThreads) void emit_pairs(const uint4* __restrict__ sdesc,
                                                           const uint32_t* __restrict__ epref,
                                                           const uint32_t* __restrict__ chunk_first,
                                                           const uint32_t* __restrict__ nvis,
                                                           const uint32_t* __restrict__ count,
                                                           const int32_t* __restrict__ status,
                                                           uint32_t* __restrict__ tkey, uint32_t* __restrict__ tval,
                                                           uint32_t* __restrict__ trec, int64_t nblk,
                                                           uint32_t* __restrict__ hist) {
  __shared__ __align__(16) uint16_t s_own[kEmitChunk];  // record that starts at the slot, then the slot's record
  __shared__ uint32_t s_wave[kEmitThreads / kWave];
  __shared__ uint32_t s_hist[kRadix];
  const uint32_t N = effective_count(nvis, status);
  const uint32_t K = effective_count(count, status);
  const int64_t nact = ((int64_t)K + kEmitChunk - 1) / kEmitChunk;
  if (N == 0 || (int64_t)blockIdx.x >= nact) return;  // uniform
  const int64_t blk = xcd_block((int64_t)blockIdx.x, nact);
  const uint32_t slot0 = (uint32_t)blk * (uint32_t)kEmitChunk;
  const uint32_t slot1 = (uint32_t)min((uint64_t)slot0 + kEmitChunk, (uint64_t)K);
  const uint32_t m0 = chunk_first[blk];
  const uint32_t m_end = slot1 < K ? chunk_first[blk + 1] + 1u : N;
  const int nr = (int)(m_end - m0);  // records that may own slots of the chunk (<= kEmitChunk + 1)
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  static_assert(kEmitItems == 8, "a thread's slots are one 16-byte word of s_own");
  uint4* own4 = (uint4*)s_own + threadIdx.x;
  *own4 = make_uint4(0u, 0u, 0u, 0u);
  if (threadIdx.x < kRadix) s_hist[threadIdx.x] = 0u;
  __syncthreads();
  for (int i = 1 + threadIdx.x; i < nr; i += kEmitThreads) {  // record 0 owns the first slot
    const uint32_t p = epref[m0 + i];
    if (p < slot1) s_own[p - slot0] = (uint16_t)i;
  }
  __syncthreads();
  {
    uint4 q = *own4;
    uint32_t x[kEmitItems] = {q.x & 0xffffu, q.x >> 16, q.y & 0xffffu, q.y >> 16,
                              q.z & 0xffffu, q.z >> 16, q.w & 0xffffu, q.w >> 16};
#pragma unroll
    for (int j = 1; j < kEmitItems; ++j) x[j] = max(x[j], x[j - 1]);
    uint32_t incl = x[kEmitItems - 1];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o, kWave);
      if (lane >= o) incl = max(incl, y);
    }
    if (lane == kWave - 1) s_wave[wave] = incl;
    uint32_t before = __shfl_up(incl, 1, kWave);
    if (lane == 0) before = 0u;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kEmitThreads / kWave; ++w) before = w < wave ? max(before, s_wave[w]) : before;
#pragma unroll
    for (int j = 0; j < kEmitItems; ++j) x[j] = max(x[j], before);
    *own4 = make_uint4(x[0] | (x[1] << 16), x[2] | (x[3] << 16), x[4] | (x[5] << 16), x[6] | (x[7] << 16));
  }
  __syncthreads();
  // four slots at a time, their descriptors in flight together
#pragma unroll
  for (int j0 = 0; j0 < kEmitItems; j0 += 4) {
    uint4 d[4];
    uint32_t p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t m = m0 + s_own[(j0 + j) * kEmitThreads + threadIdx.x];  // past slot1: the last record
      d[j] = sdesc[m];
      p[j] = epref[m];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t slot = slot0 + (j0 + j) * kEmitThreads + threadIdx.x;
      const uint32_t q = slot - p[j], w = d[j].y & 0xffffu;
      const uint32_t ty = q / w, tx = q - ty * w;
      if (slot < slot1) {
        const uint32_t tile = d[j].x + ty * (d[j].y >> 16) + tx;
        atomicAdd(&s_hist[tile & (kRadix - 1)], 1u);
        tkey[slot] = tile;
        tval[slot] = d[j].z + q;  // canonical pair index
        trec[slot] = d[j].w;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < kRadix) hist[(int64_t)threadIdx.x * nblk + blk] = s_hist[threadIdx.x];
}

template <typename KT>
__global__ __launch_bounds__(kSortThreads) void radix_hist(const KT* __restrict__ keys,
                                                           const uint32_t* __restrict__ count,
                                                           const int32_t* __restrict__ status, int shift, int64_t nblk,
                                                           uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kRadix];
  const uint32_t K = effective_count(count, status);
  const int64_t nact = ((int64_t)K + kSortTile - 1) / kSortTile;
  if ((int64_t)blockIdx.x >= nact) return;  // uniform: a column that is not read
  if (threadIdx.x < kRadix) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t blk = xcd_block((int64_t)blockIdx.x, nact);
  const int64_t base = blk * kSortTile + threadIdx.x;
  KT key[kSortItems];
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) key[k] = base + k * kSortThreads < K ? keys[base + k * kSortThreads] : KT(0);
#pragma unroll
  for (int k = 0; k < kSortItems; ++k)
    if (base + k * kSortThreads < K) atomicAdd(&h[(uint32_t)(key[k] >> shift) & (kRadix - 1)], 1u);
  __syncthreads();
  if (threadIdx.x < kRadix) hist[(int64_t)threadIdx.x * nblk + blk] = h[threadIdx.x];
}

// One block per digit: exclusive scan of that digit's counts over the first
// nact sort blocks, the ones holding keys (in place), and the digit's total.
// Each thread takes 4 consecutive columns per step of 1024.
__global__ __launch_bounds__(256) void radix_digit_scan(uint32_t* __restrict__ hist, int64_t nblk,
                                                        const uint32_t* __restrict__ count,
                                                        const int32_t* __restrict__ status,
                                                        uint32_t* __restrict__ digit_total) {
  __shared__ uint32_t s_wave[4];
  __shared__ uint32_t s_carry;
  const int64_t nact = ((int64_t)effective_count(count, status) + kSortTile - 1) / kSortTile;
  uint32_t* row = hist + (int64_t)blockIdx.x * nblk;
  if (threadIdx.x == 0) s_carry = 0;
  __syncthreads();
  for (int64_t base = 0; base < nact; base += 4 * 256) {
    const int64_t i0 = base + 4 * (int64_t)threadIdx.x;
    uint32_t x[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      x[j] = i0 + j < nact ? row[i0 + j] : 0u;
      sum += x[j];
    }
    uint32_t tot;
    uint32_t ex = block_exclusive_scan_256(sum, &tot, s_wave) + s_carry;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (i0 + j < nact) row[i0 + j] = ex;
      ex += x[j];
    }
    __syncthreads();
    if (threadIdx.x == 0) s_carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) digit_total[blockIdx.x] = s_carry;
}

// Lanes of the wave holding the same digit (among valid lanes), the digit's
// low `bits` bits alone (the others are zero in every key).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int bits) {
  uint64_t m = __ballot(valid);
  uint32_t lo = (uint32_t)m, hi = (uint32_t)(m >> 32);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    if (b >= bits) break;  // uniform
    const uint32_t t = (uint32_t)(((int32_t)(d << (31 - b))) >> 31);  // the bit, in every position
    const uint64_t bb = __ballot(t != 0u);
    lo &= ~((uint32_t)bb ^ t);
    hi &= ~((uint32_t)(bb >> 32) ^ t);
  }
  return (uint64_t)lo | ((uint64_t)hi << 32);
}

// Exclusive scan of one value per thread over the first 256 threads of the
// block (all threads call it).
__device__ __forceinline__ uint32_t exclusive_scan_first_256(uint32_t x, uint32_t* s_wave) {
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  uint32_t incl = x;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const uint32_t y = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += y;
  }
  if (lane == kWave - 1 && wave < kRadix / kWave) s_wave[wave] = incl;
  __syncthreads();
  uint32_t off = 0;
#pragma unroll
  for (int w = 0; w < kRadix / kWave; ++w) off += w < wave ? s_wave[w] : 0u;
  __syncthreads();
  return incl - x + off;
}

// One stable scatter pass for 32-bit keys; NV value arrays travel with the
// keys (NV = 1 or 2; the second may be null when NV = 1).  Each wave owns a
// contiguous eighth (512 elements) of the block's 4096 and ranks its items
// in element order against wave-private running digit counts in LDS (match
// by ballots; only the leader of a digit group updates the count), so the
// ranking needs no block barrier.  Then one barrier, per-digit prefixes over
// the waves, the elements placed in LDS in (digit, index) order, and written
// out run by run, so consecutive threads write consecutive addresses.  The
// arrays go through the same 16 KB of LDS in turn: with a buffer for each, two
// workgroups of 256 threads fitted a CU and a pass over 14.1M pairs with two
// values took 95 us (3.6 TB/s); now 78 (4.3 TB/s).
template <int NV>
__global__ __launch_bounds__(kSortThreads, 4) void radix_scatter(const uint32_t* __restrict__ kin,
                                                              const uint32_t* __restrict__ vin,
                                                              const uint32_t* __restrict__ vin2,
                                                              uint32_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                              uint32_t* __restrict__ vout2,
                                                              const uint32_t* __restrict__ count,
                                                              const int32_t* __restrict__ status, int shift, int bits,
                                                              int64_t nblk, const uint32_t* __restrict__ hist,
                                                              const uint32_t* __restrict__ digit_total) {
  constexpr int kWaves = kSortThreads / kWave;
  constexpr int kPerWave = kSortTile / kWaves;
  __shared__ uint32_t s_gbase[kRadix];  // global position of digit d's first element here, less its local position
  __shared__ uint32_t s_lbase[kRadix];  // its position within the block's digit-ordered elements
  __shared__ uint32_t s_cnt[kWaves][kRadix];  // running counts per wave, then the waves' prefixes
  __shared__ uint32_t s_wave[kWaves];
  __shared__ uint32_t s_buf[kSortTile];
  const uint32_t K = effective_count(count, status);
  const int64_t nact = ((int64_t)K + kSortTile - 1) / kSortTile;
  if ((int64_t)blockIdx.x >= nact) return;  // uniform across the block
  const int64_t blk = xcd_block((int64_t)blockIdx.x, nact);
  const int64_t base = blk * kSortTile;
  const int nvalid = (int)min((int64_t)kSortTile, (int64_t)K - base);
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = t / kWave;
#pragma unroll
  for (int q = 0; q < kWaves * kRadix / kSortThreads; ++q) (&s_cnt[0][0])[q * kSortThreads + t] = 0;
  uint32_t key[kSortItems], val[kSortItems], val2[NV == 2 ? kSortItems : 1], pos[kSortItems];
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  uint32_t* cnt = s_cnt[wave];
  const int li0 = wave * kPerWave + lane;
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) key[k] = li0 + k * kWave < nvalid ? kin[base + li0 + k * kWave] : 0u;
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) val[k] = li0 + k * kWave < nvalid ? vin[base + li0 + k * kWave] : 0u;
  if (NV == 2) {
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) val2[k] = li0 + k * kWave < nvalid ? vin2[base + li0 + k * kWave] : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) {
    const bool valid = li0 + k * kWave < nvalid;
    const uint32_t d = (key[k] >> shift) & (kRadix - 1);
    const uint64_t peers = match_digit(d, valid, bits);
    const uint32_t r = __popcll(peers & lt_mask);
    const uint32_t c = valid ? cnt[d] : 0u;  // elements of digit d earlier in this wave
    pos[k] = c + r;
    if (valid && r == 0) cnt[d] = c + (uint32_t)__popcll(peers);
    __builtin_amdgcn_wave_barrier();  // the wave's LDS updates stay in item order
  }
  __syncthreads();
  {
    // digit t: the waves' prefixes and the block's count
    uint32_t run = 0;
    if (t < kRadix) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = s_cnt[w][t];
        s_cnt[w][t] = run;
        run += c;
      }
    }
    // digit t: its elements in earlier blocks, and in all
    uint32_t before = 0, total = 0;
    if (t < kRadix) {
      const uint32_t* row = hist + (int64_t)t * nblk;
      if (digit_total) {  // uniform: rows scanned
        before = row[blk];
        total = digit_total[t];
      } else {
  #pragma unroll 8
        for (int b = 0; b < (int)nact; ++b) {
          const uint32_t c = row[b];
          before += b < (int)blk ? c : 0u;
          total += c;
        }
      }
    }
    const uint32_t lb = exclusive_scan_first_256(run, s_wave);
    const uint32_t dbase = exclusive_scan_first_256(total, s_wave);
    if (t < kRadix) {
      s_lbase[t] = lb;
      s_gbase[t] = dbase + before - lb;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) {
    const uint32_t d = (key[k] >> shift) & (kRadix - 1);
    pos[k] += s_lbase[d] + cnt[d];
    if (li0 + k * kWave < nvalid) s_buf[pos[k]] = key[k];
  }
  __syncthreads();
  uint32_t to[kSortItems];  // global position of the block's digit-ordered element t + k * kSortThreads
#pragma unroll
  for (int k = 0; k < kSortItems; ++k) {
    const int i = k * kSortThreads + t;
    const uint32_t kk = s_buf[i];
    to[k] = s_gbase[(kk >> shift) & (kRadix - 1)] + (uint32_t)i;
    if (i < nvalid) kout[to[k]] = kk;
  }
  auto move = [&](const uint32_t* v, uint32_t* out) {
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortItems; ++k)
      if (li0 + k * kWave < nvalid) s_buf[pos[k]] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortItems; ++k)
      if (k * kSortThreads + t < nvalid) out[to[k]] = s_buf[k * kSortThreads + t];
  };
  move(val, vout);
  if (NV == 2) move(val2, vout2);
}

// Per sorted pair: [start, end) of its tile's run and, if asked for, the
// 64-bit key.  Each thread takes 4 consecutive pairs (one 16-byte load; the
// key arrays are 256-byte aligned) and compares them with their neighbours.
__global__ void tile_ranges(const uint32_t* __restrict__ tkey, const uint32_t* __restrict__ ids,
                            const uint32_t* __restrict__ drec, const uint32_t* __restrict__ count,
                            const int32_t* __restrict__ status, uint64_t* __restrict__ keys,
                            uint32_t* __restrict__ ranges) {
  const uint32_t K = effective_count(count, status);
  const int64_t i0 = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (i0 >= K) return;
  uint32_t t[6];  // pairs i0 - 1 .. i0 + 4 (outside [0, K): no tile)
  if (i0 + 4 <= (int64_t)K) {
    const uint4 q = *(const uint4*)(tkey + i0);
    t[1] = q.x, t[2] = q.y, t[3] = q.z, t[4] = q.w;
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) t[1 + j] = i0 + j < (int64_t)K ? tkey[i0 + j] : 0xffffffffu;
  }
  t[0] = i0 > 0 ? tkey[i0 - 1] : 0xffffffffu;
  t[5] = i0 + 4 < (int64_t)K ? tkey[i0 + 4] : 0xffffffffu;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t i = i0 + j;
    if (i >= (int64_t)K) break;
    const uint32_t c = t[1 + j];
    if (keys) keys[i] = ((uint64_t)c << 32) | drec[ids[i]];
    if (t[j] != c) ranges[2 * (int64_t)c] = (uint32_t)i;
    if (t[2 + j] != c) ranges[2 * (int64_t)c + 1] = (uint32_t)(i + 1);
  }
}

// Heaviest-first tile schedule: tiles grouped by the bit length of their list
// length (33 groups), groups in decreasing order.  hist[0..63] counts the
// groups, hist[64..127] becomes each group's running write position.
__device__ __forceinline__ int length_group(uint32_t len) { return len ? 32 - __clz(len) : 0; }

__device__ __forceinline__ uint32_t tile_len(const uint32_t* ranges, const int32_t* status, int64_t t) {
  return *status == 0 ? ranges[2 * t + 1] - ranges[2 * t] : 0u;
}

__global__ __launch_bounds__(256) void tile_order_count(const uint32_t* __restrict__ ranges,
                                                        const int32_t* __restrict__ status, int64_t tiles,
                                                        uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[64];
  if (threadIdx.x < 64) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < tiles) atomicAdd(&h[length_group(tile_len(ranges, status, t))], 1u);
  __syncthreads();
  if (threadIdx.x < 64 && h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], h[threadIdx.x]);
}

__global__ void tile_order_scan(uint32_t* __restrict__ hist) {
  if (threadIdx.x != 0) return;
  uint32_t run = 0;
  for (int g = 63; g >= 0; --g) {
    hist[64 + g] = run;
    run += hist[g];
  }
}

__global__ __launch_bounds__(256) void tile_order_scatter(const uint32_t* __restrict__ ranges,
                                                          const int32_t* __restrict__ status, int64_t tiles,
                                                          uint32_t* __restrict__ hist, uint32_t* __restrict__ order) {
  // ranks within the block per group (LDS), one global reservation per group and block
  __shared__ uint32_t h[64], base[64];
  if (threadIdx.x < 64) h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int g = 0;
  uint32_t rank = 0;
  if (t < tiles) {
    g = length_group(tile_len(ranges, status, t));
    rank = atomicAdd(&h[g], 1u);
  }
  __syncthreads();
  if (threadIdx.x < 64 && h[threadIdx.x]) base[threadIdx.x] = atomicAdd(&hist[64 + threadIdx.x], h[threadIdx.x]);
  __syncthreads();
  if (t < tiles) order[base[g] + rank] = (uint32_t)t;
}

// Four words a thread, one store where the address allows it.
__global__ __launch_bounds__(256) void fill_u32(uint32_t* p, int64_t count, uint32_t value) {
  const int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (((uintptr_t)p & 15) == 0 && i + 4 <= count) {
    *(uint4*)(p + i) = make_uint4(value, value, value, value);
  } else {
    for (int64_t k = i; k < min(i + 4, count); ++k) p[k] = value;
  }
}

hipError_t launch_fill_u32(uint32_t* p, int64_t count, uint32_t value, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32, dim3((unsigned)((count + 1023) / 1024)), dim3(256), 0, s, p, count, value);
  return hipGetLastError();
}

// The lists' ranges and the tile schedule's counters, both zero.
__global__ __launch_bounds__(256) void clear_ranges(uint32_t* __restrict__ ranges, int64_t words,
                                                    uint32_t* __restrict__ tile_hist) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < words) ranges[i] = 0u;
  if (i < 128) tile_hist[i] = 0u;
}

// Everything up to the emission for at most 1024 ITEMS records, in one
// workgroup: pair count and capacity status, canonical offsets, the visible
// records' depth order (stable passes of 8 bits like the general path's, over
// keys that stay in LDS), their descriptors in that order with the
// output positions, and each emission chunk's first record: the same words as
// count_reduce, scan_top, compact_visible, four passes of the radix sort,
// gather_reduce, scan_top and emit_prefix leave, whose 15 launches of 2 to 8 us
// are most of a small scene's lists.  The whole call on 2000 records took 134 us
// with them and takes 52; on 8192, 152 and 72 (112 by the general path); on
// 12000, 152 and 89 (110).  At 12 records a thread its one workgroup is a match
// for the general path at some 15 thousand; at 20 it spills and loses.
constexpr int kSmallThreads = 1024;
constexpr int64_t small_records(int items) { return (int64_t)kSmallThreads * items; }

template <int ITEMS>
__global__ __launch_bounds__(kSmallThreads) void small_lists(const float4* __restrict__ splats,
                                                             const uint32_t* __restrict__ tt, int nrec, int64_t n,
                                                             ViewTable vt, float inv_tw, float inv_th,
                                                             uint64_t capacity, uint32_t* __restrict__ count,
                                                             uint32_t* __restrict__ nvis,
                                                             int32_t* __restrict__ status,
                                                             uint32_t* __restrict__ offsets, uint4* desc,
                                                             uint4* __restrict__ sdesc, uint32_t* __restrict__ epref,
                                                             uint32_t* __restrict__ chunk_first,
                                                             uint32_t* __restrict__ drec) {
  constexpr int kWaves = kSmallThreads / kWave;
  __shared__ uint32_t s_key[kSmallThreads * ITEMS];
  __shared__ uint16_t s_idx[kSmallThreads * ITEMS];
  __shared__ uint16_t s_cnt[kWaves][kRadix];
  __shared__ uint32_t s_base[kRadix];
  __shared__ uint32_t s_wave[kWaves];
  __shared__ uint2 s_part[ITEMS * kWaves];  // per slice and wave: pairs, visible records; then their scans
  __shared__ unsigned long long s_pairs[kWaves];
  __shared__ uint32_t s_diff;
  const int t = threadIdx.x, lane = t & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const uint64_t lt_mask = (1ull << lane) - 1ull;
  // slices of 1024 consecutive records
  uint32_t c[ITEMS], ex[ITEMS], vx[ITEMS];
  unsigned long long sum = 0;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) c[j] = j * kSmallThreads + t < nrec ? tt[j * kSmallThreads + t] : 0u;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const uint32_t incl = wave_inclusive_sum(c[j]);
    const uint64_t vis = __ballot(c[j] != 0u);
    ex[j] = incl - c[j];
    vx[j] = (uint32_t)__popcll(vis & lt_mask);
    sum += c[j];
    if (lane == kWave - 1) s_part[j * kWaves + wave] = make_uint2(incl, (uint32_t)__popcll(vis));
  }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) sum += __shfl_xor(sum, o, kWave);
  if (lane == 0) s_pairs[wave] = sum;
  if (t == 0) s_diff = 0u;
  __syncthreads();
  constexpr int kParts = ITEMS * kWaves / kWave;  // of a lane
  static_assert(kParts * kWave == ITEMS * kWaves, "whole lanes");
  if (wave == 0) {
    uint2 a[kParts];
    uint32_t x = 0, y = 0;
#pragma unroll
    for (int k = 0; k < kParts; ++k) a[k] = s_part[kParts * lane + k], x += a[k].x, y += a[k].y;
    uint32_t px = wave_inclusive_sum(x) - x, py = wave_inclusive_sum(y) - y;
#pragma unroll
    for (int k = 0; k < kParts; ++k) {
      s_part[kParts * lane + k] = make_uint2(px, py);
      px += a[k].x;
      py += a[k].y;
    }
    if (lane == kWave - 1) s_base[0] = py;
  }
  unsigned long long K = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) K += s_pairs[w];
  __syncthreads();
  const int N = (int)s_base[0];
  if (t == 0) {
    *count = K > 0xffffffffull ? 0xffffffffu : (uint32_t)K;
    *nvis = (uint32_t)N;
    *status = K > (unsigned long long)capacity ? 1 : 0;
  }
  if (K > (unsigned long long)capacity) return;  // overflow: no lists this step (uniform)
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int r = j * kSmallThreads + t;
    const uint2 part = s_part[j * kWaves + wave];
    ex[j] += part.x;
    vx[j] += part.y;
    if (r < nrec) offsets[r] = ex[j];
    if (c[j] == 0u) continue;
    const float2 uv = *(const float2*)(splats + (int64_t)r * 3);            // u, v
    const float2 rd = *((const float2*)(splats + (int64_t)r * 3 + 1) + 1);  // radius, depth
    int v = 0;
    while (v + 1 < vt.nviews && r >= (int64_t)(v + 1) * n) ++v;
    const ViewArgs& va = vt.v[v];
    int x0, y0, x1, y1;
    tile_rect(uv.x, uv.y, rd.x, inv_tw, inv_th, va.TX, va.TY, &x0, &y0, &x1, &y1);
    const uint32_t dbits = __float_as_uint(rd.y);  // depth > near plane > 0: bits order as values
    s_key[vx[j]] = dbits;
    s_idx[vx[j]] = (uint16_t)vx[j];
    desc[vx[j]] = make_uint4((uint32_t)(va.tile_off + y0 * va.TX + x0),
                             (uint32_t)(x1 - x0 + 1) | ((uint32_t)va.TX << 16), ex[j], (uint32_t)r);
    if (drec) drec[r] = dbits;
  }
  __syncthreads();
  if (N == 0) return;  // uniform
  // Each wave owns the positions [wave R 64, (wave + 1) R 64), R of at most ITEMS rounds.
  const int R = (N + kSmallThreads - 1) / kSmallThreads;
  const int p0 = wave * R * kWave + lane;
  uint32_t key[ITEMS], idx[ITEMS], pos[ITEMS];
  {  // the bits in which any two keys differ: a pass over equal digits moves nothing
    uint32_t diff = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
      if (j < R && p0 + j * kWave < N) diff |= s_key[p0 + j * kWave] ^ s_key[0];
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) diff |= __shfl_xor(diff, o, kWave);
    if (lane == 0 && diff != 0u) atomicOr(&s_diff, diff);
  }
  __syncthreads();
  const uint32_t diff = s_diff;
#pragma unroll 1
  for (int shift = 0; shift < 32; shift += 8) {
    if (((diff >> shift) & (kRadix - 1)) == 0u) continue;  // uniform
#pragma unroll
    for (int q = 0; q < kWaves * kRadix / 2 / kSmallThreads; ++q) ((uint32_t*)s_cnt)[q * kSmallThreads + t] = 0u;
    uint16_t* cnt = s_cnt[wave];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const bool valid = j < R && p0 + j * kWave < N;
      key[j] = valid ? s_key[p0 + j * kWave] : 0u;
      idx[j] = valid ? s_idx[p0 + j * kWave] : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j >= R) break;  // uniform
      const bool valid = p0 + j * kWave < N;
      const uint32_t d = (key[j] >> shift) & (kRadix - 1);
      const uint64_t peers = match_digit(d, valid, 8);
      const uint32_t r = (uint32_t)__popcll(peers & lt_mask);
      const uint32_t k = valid ? cnt[d] : 0u;  // elements of digit d earlier in this wave
      pos[j] = k + r;
      if (valid && r == 0) cnt[d] = (uint16_t)(k + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();  // the wave's LDS updates stay in item order
    }
    __syncthreads();
    uint32_t run = 0;
    if (t < kRadix) {
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t k = s_cnt[w][t];
        s_cnt[w][t] = (uint16_t)run;
        run += k;
      }
    }
    const uint32_t lb = exclusive_scan_first_256(run, s_wave);
    if (t < kRadix) s_base[t] = lb;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j >= R || p0 + j * kWave >= N) continue;
      const uint32_t d = (key[j] >> shift) & (kRadix - 1);
      const uint32_t to = s_base[d] + cnt[d] + pos[j];
      s_key[to] = key[j];
      s_idx[to] = (uint16_t)idx[j];
    }
    __syncthreads();
  }
  // depth order: descriptors, output positions, the chunks' first records
  uint4 d[ITEMS];
  uint32_t run = 0;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    d[j] = j < R && p0 + j * kWave < N ? desc[s_idx[p0 + j * kWave]] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    c[j] = j < R && p0 + j * kWave < N ? tt[d[j].w] : 0u;
  }
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const uint32_t incl = wave_inclusive_sum(c[j]);
    ex[j] = run + incl - c[j];
    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  }
  if (lane == 0) s_wave[wave] = run;
  __syncthreads();
  uint32_t off = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) off += w < wave ? s_wave[w] : 0u;
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    const int m = p0 + j * kWave;
    if (j >= R || m >= N) continue;
    const uint32_t e = off + ex[j];
    sdesc[m] = d[j];
    epref[m] = e;
    // chunks whose first position lies in [e, e + c)
    for (uint64_t q = ((uint64_t)e + kEmitChunk - 1) / kEmitChunk; q * kEmitChunk < (uint64_t)e + c[j]; ++q)
      chunk_first[q] = (uint32_t)m;
  }
}

static inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct SortWs {
  uint2* block_sums;        // [record blocks] pairs and visible records per block, then their scans
  uint2* eblock_sums;       // [emission scan blocks] pairs per block of depth-sorted records, then their scan
  uint32_t* nvis;           // [1] number of visible records
  uint32_t* dkey;           // [nrec] depth bits of the visible records
  uint32_t* dval;           // [nrec] their compact indices
  uint32_t* dkey_alt;
  uint32_t* dval_alt;
  uint4* desc;              // [nrec] emission descriptors of the visible records (compact index)
  uint4* sdesc;             // [nrec] the same in depth order
  uint32_t* drec;           // [nrec] depth bits by record (for the keys)
  uint32_t* tkey;           // [capacity] tile id of each pair
  uint32_t* tkey_alt;
  uint32_t* tval_alt;       // [capacity] canonical pair index (second buffer)
  uint32_t* trec_alt;       // [capacity] record id (second buffer)
  uint32_t* hist;           // [256][sort blocks]
  uint32_t* digit_total;    // [256]
  uint32_t* tile_hist;      // [128] tile schedule counters
  uint32_t* chunk_first;    // [capacity / kEmitChunk + 1] first record of each emission chunk
  size_t bytes;
};

static SortWs carve(const SortPlan& p, uint64_t capacity, void* ws) {
  SortWs w{};
  char* b = (char*)ws;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    uint32_t* q = (uint32_t*)(b + o);
    o += align256(bytes);
    return q;
  };
  const size_t nb = (size_t)p.scan_blocks, nrec = (size_t)p.nrec;
  w.block_sums = (uint2*)take(8 * (size_t)p.rec_blocks);
  w.eblock_sums = (uint2*)take(8 * nb);
  w.nvis = take(8);  // [0] visible records, [1] their pairs (unused)
  w.dkey = take(4 * nrec);
  w.dval = take(4 * nrec);
  w.dkey_alt = take(4 * nrec);
  w.dval_alt = take(4 * nrec);
  w.desc = (uint4*)take(16 * nrec);
  w.sdesc = (uint4*)take(16 * nrec);
  w.drec = take(4 * nrec);
  w.tkey = take(4 * (size_t)capacity);
  w.tkey_alt = take(4 * (size_t)capacity);
  w.tval_alt = take(4 * (size_t)capacity);
  w.trec_alt = take(4 * (size_t)capacity);
  w.hist = take(4 * (size_t)kRadix * (size_t)(p.sort_blocks > p.rec_sort_blocks ? p.sort_blocks : p.rec_sort_blocks));
  w.digit_total = take(4 * (size_t)kRadix);
  w.tile_hist = take(4 * 128);
  w.chunk_first = take(4 * ((size_t)capacity / kEmitChunk + 2));
  w.bytes = o;
  return w;
}

size_t bin_sort_ws_bytes(const SortPlan& p) { return carve(p, p.capacity, nullptr).bytes; }

// One stable LSD pass per 8 key bits; the result lands back in (k0, v0, u0)
// when the number of passes is even and in (k1, v1, u1) when it is odd.
// counted: the first pass's histogram is there.
template <typename KT, int NV>
static void radix_sort(KT* k0, uint32_t* v0, uint32_t* u0, KT* k1, uint32_t* v1, uint32_t* u1, int key_bits,
                       const uint32_t* count, const int32_t* status, int64_t nblk, bool counted, const SortWs& w,
                       hipStream_t s) {
  KT* kb[2] = {k0, k1};
  uint32_t* vb[2] = {v0, v1};
  uint32_t* ub[2] = {u0, u1};
  int cur = 0;
  for (int shift = 0; shift < key_bits && nblk > 0; shift += 8) {
    const int bits = key_bits - shift < 8 ? key_bits - shift : 8;
    if (shift > 0 || !counted)
      hipLaunchKernelGGL((radix_hist<KT>), dim3((unsigned)nblk), dim3(kSortThreads), 0, s, kb[cur], count, status,
                         shift, nblk, w.hist);
    // up to kScanBlocks blocks, each sums the rows of the histogram itself
    uint32_t* totals = nblk > kScanBlocks ? w.digit_total : nullptr;
    if (totals)
      hipLaunchKernelGGL(radix_digit_scan, dim3(kRadix), dim3(256), 0, s, w.hist, nblk, count, status, totals);
    hipLaunchKernelGGL((radix_scatter<NV>), dim3((unsigned)nblk), dim3(kSortThreads), 0, s, kb[cur], vb[cur],
                       ub[cur], kb[cur ^ 1], vb[cur ^ 1], ub[cur ^ 1], count, status, shift, bits, nblk, w.hist,
                       totals);
    cur ^= 1;
  }
}

hipError_t launch_bin_sort(const SortPlan& plan, const float4* splats, const uint32_t* tiles_touched, int64_t n,
                           const ViewTable& vt, float inv_tw, float inv_th, const BinOut& out, uint64_t capacity,
                           void* ws, hipStream_t s) {
  const SortWs w = carve(plan, capacity, ws);
  const int64_t words = 2 * (int64_t)vt.total_tiles;
  if (words > 0)
    hipLaunchKernelGGL(clear_ranges, dim3((unsigned)(((words > 128 ? words : 128) + 255) / 256)), dim3(256), 0, s,
                       out.ranges, words, w.tile_hist);
  const int64_t nb = plan.scan_blocks;
  uint32_t* count = out.count;
  int32_t* status = out.status;
  const int64_t rb = plan.rec_blocks;
  // one workgroup is faster than the launches it saves up to here (see small_lists)
  const bool small = nb > 0 && plan.nrec <= small_records(12);
  if (rb > 0 && !small)
    hipLaunchKernelGGL(count_reduce, dim3((unsigned)rb), dim3(kScanThreads), 0, s, tiles_touched, plan.nrec,
                       w.block_sums);
  // K and the capacity status, and the number of visible records
  if (!small)
    hipLaunchKernelGGL(scan_top, dim3(1), dim3(1024), 0, s, w.block_sums, rb, (const uint32_t*)nullptr,
                       capacity, count, w.nvis, status);
  if (nb > 0) {
    // the emission's positions go to dkey_alt, free after the depth sort
    uint32_t* epref = w.dkey_alt;
    if (small) {
      hipLaunchKernelGGL(plan.nrec <= small_records(8) ? small_lists<8> : small_lists<12>, dim3(1), dim3(kSmallThreads),
                         0, s, splats, tiles_touched, (int)plan.nrec, n, vt, inv_tw, inv_th, capacity, count, w.nvis,
                         status, out.offsets, w.desc, w.sdesc, epref, w.chunk_first,
                         out.keys ? w.drec : (uint32_t*)nullptr);
    } else {
      hipLaunchKernelGGL(compact_visible, dim3((unsigned)rb), dim3(kScanThreads), 0, s, splats, tiles_touched,
                         plan.nrec, n, vt, inv_tw, inv_th, w.block_sums, status, out.offsets, w.dkey, w.dval, w.desc,
                         out.keys ? w.drec : (uint32_t*)nullptr);
      // depth order of the visible records (four passes: the result is back in dkey/dval)
      radix_sort<uint32_t, 1>(w.dkey, w.dval, nullptr, w.dkey_alt, w.dval_alt, nullptr, 32, w.nvis, status,
                              plan.rec_sort_blocks, false, w, s);
      hipLaunchKernelGGL(gather_reduce, dim3((unsigned)nb), dim3(kScanThreads), 0, s, w.desc, w.dval, w.nvis, status,
                         vt, w.sdesc, epref, w.eblock_sums);
      hipLaunchKernelGGL(scan_top, dim3(1), dim3(1024), 0, s, w.eblock_sums, nb, w.nvis, (uint64_t)0,
                         w.nvis + 1, (uint32_t*)nullptr, (int32_t*)nullptr);  // total unused (equals K)
      hipLaunchKernelGGL(emit_prefix, dim3((unsigned)nb), dim3(kScanThreads), 0, s, w.nvis, count, w.eblock_sums, status,
                         epref, w.chunk_first);
    }
    // emit so that the tile sort ends in (tkey, pair_index, ids)
    const bool even = (plan.tile_bits + 7) / 8 % 2 == 0;
    const int64_t emit_blocks = ((int64_t)capacity + kEmitChunk - 1) / kEmitChunk;
    if (emit_blocks > 0)
      hipLaunchKernelGGL(emit_pairs, dim3((unsigned)emit_blocks), dim3(kEmitThreads), 0, s, w.sdesc, epref,
                         w.chunk_first, w.nvis, count, status, even ? w.tkey : w.tkey_alt,
                         even ? out.pair_index : w.tval_alt, even ? out.ids : w.trec_alt, plan.sort_blocks, w.hist);
    if (even)
      radix_sort<uint32_t, 2>(w.tkey, out.pair_index, out.ids, w.tkey_alt, w.tval_alt, w.trec_alt, plan.tile_bits,
                              count, status, plan.sort_blocks, true, w, s);
    else
      radix_sort<uint32_t, 2>(w.tkey_alt, w.tval_alt, w.trec_alt, w.tkey, out.pair_index, out.ids, plan.tile_bits,
                              count, status, plan.sort_blocks, true, w, s);
  }
  const int64_t cap_blocks = ((int64_t)capacity + 1023) / 1024;
  if (cap_blocks > 0 && nb > 0)
    hipLaunchKernelGGL(tile_ranges, dim3((unsigned)cap_blocks), dim3(256), 0, s, w.tkey, out.ids, w.drec, count,
                       status, out.keys, out.ranges);
  if (out.order && vt.total_tiles > 0) {
    const int64_t T = vt.total_tiles;
    const unsigned tb = (unsigned)((T + 255) / 256);
    hipLaunchKernelGGL(tile_order_count, dim3(tb), dim3(256), 0, s, out.ranges, status, T, w.tile_hist);
    hipLaunchKernelGGL(tile_order_scan, dim3(1), dim3(64), 0, s, w.tile_hist);
    hipLaunchKernelGGL(tile_order_scatter, dim3(tb), dim3(256), 0, s, out.ranges, status, T, w.tile_hist, out.order);
  }
  return hipGetLastError();
}

}  // namespace gs
