// Internal declarations shared by the HIP translation units of liboctgs.
// Written for gfx950 (CDNA4): 64-lane wavefronts, 256-thread blocks of four
// waves, MFMA for the decode GEMMs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>
#include <cmath>
#include <cstring>

#include "../../include/octgs.h"

namespace octgs {

constexpr int kWave = 64;
constexpr int kBlock = 256;          // threads per block in every kernel
constexpr int kTile = 16;            // screen tile edge in pixels
constexpr int kChunk = 1024;         // elements per block in the two-pass compactions
constexpr int kChunkPerThread = kChunk / kBlock;  // 4
constexpr int kGroups = kChunk / 64;              // 64-element ballot groups per block
constexpr int kGaussFields = 14;
constexpr int kProjVec = 3;          // float4 records per projected Gaussian
constexpr int kMaxK = 16;

// FP32 -> BF16 bit pattern, round to nearest even (NaN kept quiet): one
// v_cvt_pk_bf16_f32, which gives what the integer arithmetic for it (five
// instructions) gives for all 2^32 inputs.
__device__ __forceinline__ uint16_t f2bf(float f) {
  return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// ---------------------------------------------------------------------------
// wave64 helpers
// ---------------------------------------------------------------------------

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t lanemask_lt() {
  int l = __lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

__device__ __forceinline__ uint64_t ballot(int pred) { return __ballot(pred); }

// v plus the DPP-moved v of the rows in ROWMASK (lanes the move does not reach
// add 0).
template <int CTRL, int ROWMASK>
__device__ __forceinline__ uint32_t dpp_add(uint32_t v) {
  return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWMASK, 0xF, true);
}

// Inclusive prefix sum across the 64 lanes of a wave, by DPP alone: shifts by
// 1, 2, 4 and 8 within each 16-lane row, then the last lane of rows 0 and 2
// into rows 1 and 3, then lane 31 into rows 2 and 3 (shuffles through LDS cost
// six dependent round trips).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v = dpp_add<0x111, 0xF>(v);
  v = dpp_add<0x112, 0xF>(v);
  v = dpp_add<0x114, 0xF>(v);
  v = dpp_add<0x118, 0xF>(v);
  v = dpp_add<0x142, 0xA>(v);
  return dpp_add<0x143, 0xC>(v);
}

// Cross-lane moves without LDS: DPP within 16-lane rows, permlane swaps
// across rows (gfx950).  Controls: quad_perm [1,0,3,2] = lane ^ 1, quad_perm
// [2,3,0,1] = lane ^ 2, row_half_mirror = 7 - lane within 8, row_ror:8 =
// lane ^ 8 within 16.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppRor8 = 0x128;

// (x, y) -> (x with rows 1, 3 replaced by y's rows 0, 2; y with rows 0, 2
// replaced by x's rows 1, 3): x + y sums lanes L and L ^ 16, keeping x's
// value in rows 0 and 2 and y's in rows 1 and 3.
__device__ __forceinline__ void swap16(uint32_t &x, uint32_t &y) {
  const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
  x = r[0];
  y = r[1];
}
// The same across halves: x + y sums lanes L and L ^ 32, x's value in the
// lower half and y's in the upper.
__device__ __forceinline__ void swap32(uint32_t &x, uint32_t &y) {
  const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  x = r[0];
  y = r[1];
}

// Sum over the wave, the same bits in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
  v += dpp_u<kDppXor1>(v);
  v += dpp_u<kDppXor2>(v);
  v += dpp_u<kDppHalfMirror>(v);
  v += dpp_u<kDppRor8>(v);
  uint32_t x = v, y = v;
  swap16(x, y);
  v = x + y;
  x = v; y = v;
  swap32(x, y);
  return x + y;
}

__device__ __forceinline__ float wave_sum_f(float v) {
  v += __uint_as_float(dpp_u<kDppXor1>(__float_as_uint(v)));
  v += __uint_as_float(dpp_u<kDppXor2>(__float_as_uint(v)));
  v += __uint_as_float(dpp_u<kDppHalfMirror>(__float_as_uint(v)));
  v += __uint_as_float(dpp_u<kDppRor8>(__float_as_uint(v)));
  uint32_t x = __float_as_uint(v), y = x;
  swap16(x, y);
  v = __uint_as_float(x) + __uint_as_float(y);
  x = __float_as_uint(v); y = x;
  swap32(x, y);
  return __uint_as_float(x) + __uint_as_float(y);
}

// Sum of v over the 256 threads of a block, returned to thread 0 (LDS
// scratch of 4 floats).
__device__ __forceinline__ float block_sum_f(float v, float *red) {
  v = wave_sum_f(v);
  if (__lane_id() == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}

// Sum of a[0..b) by the 256 threads of a block, returned per thread
// (partial sums; the caller reduces).  Loads are unconditional at a clamped
// index, four per thread per step, so they are in flight together.
__device__ __forceinline__ uint32_t partial_sum_prefix(const uint32_t *a, int b) {
  uint32_t s = 0;
  const int t = threadIdx.x;
  for (int i0 = 0; i0 < b; i0 += 4 * kBlock) {
    uint32_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = a[min(i0 + u * kBlock + t, b - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) s += i0 + u * kBlock + t < b ? v[u] : 0u;
  }
  return s;
}

// Relaxed device-scope (all XCDs) atomics for look-back status words.
__device__ __forceinline__ uint32_t ld_acq(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_rel(uint32_t *p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tile scheduling of the per-tile kernels (one block per tile).  Blocks are
// dealt round-robin over the 8 XCDs, so block b runs on XCD b % 8.  Tiles
// are grouped in squares of kTileGroup x kTileGroup and group g goes to XCD
// g % 8: every XCD gets groups from all over the image, which balances the
// dense and sparse regions of a view across the XCDs, while the tiles of one
// group, which share most of their Gaussians, stay in one L2.  On request
// (OCTGS_RASTER_TILE_ORDER) the rasterizer then orders each XCD's tiles by
// list length, longest first (order_tiles), so its last blocks are short.
constexpr uint32_t kXcds = 8;
constexpr uint32_t kTileGroup = 4;
// Largest number of 16x16 tiles per image (about 4.3 gigapixels): tile ids,
// sort keys and the per-tile grids stay well inside 32 bits.
constexpr int64_t kMaxTiles = int64_t(1) << 24;
inline bool image_tiles_ok(int32_t width, int32_t height) {
  if (width <= 0 || height <= 0) return false;
  return (int64_t)((width + 15) / 16) * ((height + 15) / 16) <= kMaxTiles;
}

// Blocks to launch: 8 x kTileGroup^2 x ceil(groups / 8); the blocks past the
// last group and those on tiles outside a partial edge group exit at once.
__host__ __device__ inline uint32_t tile_grid_blocks(int tiles_x, int tiles_y) {
  const uint32_t gx = (tiles_x + kTileGroup - 1) / kTileGroup;
  const uint32_t gy = (tiles_y + kTileGroup - 1) / kTileGroup;
  return (gx * gy + kXcds - 1) / kXcds * kXcds * kTileGroup * kTileGroup;
}

// The tile of block bid, or -1 for a block without one.  A bijection from
// the blocks that have a tile onto the tiles.
__device__ __forceinline__ int32_t tile_of_block(uint32_t bid, int tiles_x, int tiles_y) {
  const uint32_t gx = (tiles_x + kTileGroup - 1) / kTileGroup;
  const uint32_t gy = (tiles_y + kTileGroup - 1) / kTileGroup;
  const uint32_t xcd = bid % kXcds, slot = bid / kXcds;
  const uint32_t g = xcd + kXcds * (slot / (kTileGroup * kTileGroup));
  const uint32_t w = slot % (kTileGroup * kTileGroup);
  if (g >= gx * gy) return -1;
  const uint32_t tx = (g % gx) * kTileGroup + w % kTileGroup;
  const uint32_t ty = (g / gx) * kTileGroup + w / kTileGroup;
  if (tx >= (uint32_t)tiles_x || ty >= (uint32_t)tiles_y) return -1;
  return (int32_t)(ty * (uint32_t)tiles_x + tx);
}

// ---------------------------------------------------------------------------
// rasterizer workspace
// ---------------------------------------------------------------------------

struct RasterHeader {
  uint32_t n_slots, n_visible, n_pairs, pair_overflow, sync_error;
  uint32_t n_candidates;  // rectangle tiles of the survivors (saturated at kLbVal)
  uint32_t n_emit;        // training: pair numbers handed out (holes of huge rectangles included)
  uint32_t n_listed;      // pairs in the sorted list (n_pairs, or 0 on overflow)
  uint32_t tile_ordered;  // 1 if the forward wrote tile_order (OCTGS_RASTER_TILE_ORDER)
  uint32_t scan_ticket;   // tile scan: block numbers in the order blocks start
  uint32_t bin_cursor;    // bin-list entries handed out
  uint32_t n_over;        // bins whose list is longer than one block sorts (kBinCap)
  uint32_t n_slices;      // and the slices of their depths
  uint32_t copy_next, copy_done;    // their entries' copy and the slices: units handed out,
  uint32_t slice_next, slice_done;  // and units done
  uint32_t reserved[15];
};

// Screen bins: rectangles of 2^sx x 2^sy tiles (at most 32, one mask bit per
// tile).  A Gaussian is handed to the bins its rectangle meets, each bin's
// list is put into depth order by one block, and the bin's tiles take their
// entries from the ordered list.
struct BinGrid {
  int32_t sx, sy;        // log2 of the bin's size in tiles
  int32_t nx, ny;        // bins of the image
  int32_t gx;            // bin columns that a rectangle (16-bit tile coordinates) can reach
  int32_t band_rows;     // bin rows that one grouping pass covers (all, but for huge images)
};

constexpr int kSlots = 512;                       // Gaussian slots per projection block
constexpr uint32_t kGroupBins = 16;               // bins that a survivor hands itself to directly
constexpr uint32_t kGroupBinsFull = 4;            // ... where the block's would not fit its stretch
constexpr uint32_t kGroupWords = 3u * kGroupBinsFull * kSlots;  // a block's stretch of the groups
constexpr uint32_t kTilesUnknown = ~0u;
constexpr uint32_t kKeepBits = 64;                // rectangle tiles that a slot's keep mask holds
constexpr int kMaxBandBins = 8192;                // bins of one grouping pass
constexpr int kMaxTileCoord = 65535;              // tiles past this column or row list nothing
constexpr int kBinThreads = 512;
constexpr int kBinItems = 8;
constexpr int kBinCap = kBinThreads * kBinItems;  // longest list that one block sorts at once
constexpr int kScanThreads = 512, kScanTiles = 16;  // tile scan: threads, tiles per thread
constexpr uint32_t kCopyCap = 16384;              // longest list that its bin's block copies by itself
constexpr uint32_t kLongSeg = 8;                  // fewest slot blocks of a unit that copies a long bin
constexpr uint32_t kSliceRow = 36;                // words per slice: bin, index, start, entries, tiles
// Slices of a bin of m > kBinCap entries: 1,536 each on average, so that few are
// more than the 2,048 that four entries per thread sort.
constexpr uint32_t kSliceEntries = 1536;
__host__ __device__ inline uint32_t long_slices(uint32_t m) { return (m + kSliceEntries - 1) / kSliceEntries; }
constexpr int kPairRow = 10;                      // words per pair of gpair: 9 gradients, slot

struct RasterWs {
  RasterHeader *hdr;
  uint64_t *vis_mask;     // [gcap / 64]
  uint32_t *blk_vis;      // [nblk_g] survivors of each block of kSlots slots
  uint32_t *blk_cand;     // [nblk_g] their rectangle tiles (saturated at kLbVal)
  uint32_t *blk_large;    // [nblk_g] large survivors in the block's group
  uint32_t *blk_pairs;    // [nblk_g] training: pair numbers of the block, then their prefix
  float4 *proj;           // [gcap][3]: (mx, my, A, B) (C, log2 opacity, r, g) (b, qa, qb, qc);
                          // A, B, C = conic scaled for exp2: -0.5 log2e ca, -log2e cb, -0.5 log2e cc;
                          // qa, qb, qc = the conic itself (tile test)
  ulonglong2 *rect;       // [gcap] x: packed u16 x0, y0, x1, y1; y: kept tiles of the rectangle,
                          // row-major, where it has at most kKeepBits (else unused)
  uint32_t *pair_base;    // [gcap] training: first pair number of the slot within its block's
                          // (slot_block)
  uint16_t *group_off;    // [nblk_g][group_pitch] start of each bin's entries in the block's group
  uint32_t *group;        // [nblk_g][kGroupWords] from the front, grouped by bin: depth key, slot,
                          // the bin's tiles that it is listed in (kTilesUnknown: to be tested);
                          // from the back the large survivors, over more bins than that:
                          // rectangle (2 words), depth key, slot; every bin looks through these
  uint2 *bin_range;       // [bins] start and length of the bin's list
  uint32_t *bin_slot[2];  // [pcap] bin lists in depth order: slots ([0]: long lists before they
                          // are sorted, [1]: after)
  uint32_t *bin_mask[2];  // [pcap] and the bin's tiles that each is listed in
  uint32_t *over_bin;     // [pcap / kBinCap + 1][2] bins with longer lists, entries copied
  uint32_t *slices;       // [long_slices of all of them][kSliceRow]
  uint32_t *tile_count;   // [tiles], padded to whole scan blocks (in tile_order's place)
  uint32_t *lb_scan;      // [scan blocks] look-back status of the tile scan
  uint32_t *tkey;         // [pcap] tile of each listed pair, in list order (bin keys of long
                          // lists before)
  uint32_t *tval;         // [pcap] its slot
  uint32_t *ranges;       // [tiles][2]
  uint32_t *tile_order;   // [tile_grid_blocks] tile of each compositing block (~0u: none),
                          // written only with OCTGS_RASTER_TILE_ORDER
  float *dproj;           // [gcap][9] backward: d(mx, my, ca, cb, cc, opacity, r, g, b)
  float *gpair;           // [pcap][kPairRow] backward: the same per pair number, then the slot
  float *chunk_part;      // [ceil(pcap / 64)][2][9] backward: sums of a 64-pair chunk's first and
                          // last run where the run crosses the chunk's start or end
  BinGrid bins;
  int64_t gcap, pcap;
  int32_t tiles_x, tiles_y, nblk_g, group_pitch, scan_blocks;
  float xmax, ymax;            // last pixel centre of the image: W - 0.5, H - 0.5
  size_t bytes;
};

// Tile test, canonical FP32: does the 3-sigma ellipse q(p) <= 9,
// q = qa dx^2 + 2 qb dx dy + qc dy^2 around (mx, my), meet the box of the
// tile's pixel centres inside the image, [16 tx + 0.5, min(16 tx + 15.5,
// W - 0.5)] x [16 ty + 0.5, min(16 ty + 15.5, H - 0.5)]?  (Pixels of a
// partial edge tile past the image are not drawn, so they do not list a
// Gaussian.)  The convex quadratic's minimum over the box is 0 with the mean
// inside; otherwise it lies on an edge facing the mean, at the 1D minimiser
// clamped to the edge:
//   X0 = (float)(16 tx) + 0.5, X1 = fminf(X0 + 15, xmax) (Y alike)
//   mean's x outside [X0, X1]: xe = nearer of X0, X1; dx = xe - mx;
//     ys = min(max(my - (qb * dx) / qc, Y0), Y1); dy = ys - my;
//     q1 = fmaf(qa * dx, dx, fmaf(2 * qb * dx, dy, qc * dy * dy))
//   mean's y outside [Y0, Y1]: the same with the roles of x and y swapped
//   keep iff min(q1, q2) <= 9.
__device__ __forceinline__ bool tile_meets_ellipse(float mx, float my, float qa, float qb, float qc,
                                                   uint32_t tx, uint32_t ty, float xmax,
                                                   float ymax) {
  const float X0 = (float)(16u * tx) + 0.5f, X1 = fminf(X0 + 15.0f, xmax);
  const float Y0 = (float)(16u * ty) + 0.5f, Y1 = fminf(Y0 + 15.0f, ymax);
  const bool in_x = !(mx < X0) && !(mx > X1), in_y = !(my < Y0) && !(my > Y1);
  float q = INFINITY;
  if (!in_x) {
    const float xe = mx < X0 ? X0 : X1;
    const float dx = xe - mx;
    const float ys = fminf(fmaxf(my - (qb * dx) / qc, Y0), Y1);
    const float dy = ys - my;
    q = __builtin_fmaf(qa * dx, dx, __builtin_fmaf(2.0f * qb * dx, dy, qc * dy * dy));
  }
  if (!in_y) {
    const float ye = my < Y0 ? Y0 : Y1;
    const float dy = ye - my;
    const float xs = fminf(fmaxf(mx - (qb * dy) / qa, X0), X1);
    const float dx = xs - mx;
    q = fminf(q, __builtin_fmaf(qa * dx, dx, __builtin_fmaf(2.0f * qb * dx, dy, qc * dy * dy)));
  }
  return (in_x && in_y) || q <= 9.0f;
}

// (x0, y0, x1, y1) of a packed rectangle, tiles, end exclusive.
struct TileRect {
  uint32_t x0, y0, x1, y1;
};
__device__ __forceinline__ uint64_t pack_rect(int x0, int y0, int x1, int y1) {
  return (uint64_t)(uint16_t)x0 | ((uint64_t)(uint16_t)y0 << 16) | ((uint64_t)(uint16_t)x1 << 32) |
         ((uint64_t)(uint16_t)y1 << 48);
}
__device__ __forceinline__ TileRect unpack_rect(uint64_t r) {
  return TileRect{(uint32_t)(r & 0xffff), (uint32_t)((r >> 16) & 0xffff),
                  (uint32_t)((r >> 32) & 0xffff), (uint32_t)(r >> 48)};
}
__device__ __forceinline__ uint32_t rect_tiles(const TileRect &r) {
  return (r.x1 - r.x0) * (r.y1 - r.y0);
}

// Blocks of slots in use by a view of n slots, and the block that projects a
// slot: waves of 64 consecutive slots are dealt over the blocks in turn, since
// neighbouring slots are of one octree level and their rectangles of one size.
__host__ __device__ inline uint32_t slot_blocks(uint32_t n) { return (n + kSlots - 1) / kSlots; }
__device__ __forceinline__ uint32_t slot_block(uint32_t slot, uint32_t nblk) {
  return (slot / kWave) % nblk;
}

// First pair number of a slot's pairs, and of its tile (tx, ty): the tile's
// rank among the kept tiles of the rectangle (row-major), or, where it has more
// than kKeepBits tiles, its place among all of them.
__device__ __forceinline__ uint32_t pair_rank(const TileRect &r, uint64_t keep, uint32_t tx,
                                              uint32_t ty) {
  const uint32_t loc = (ty - r.y0) * (r.x1 - r.x0) + (tx - r.x0);
  return rect_tiles(r) > kKeepBits ? loc
                                   : (uint32_t)__popcll(keep & ((1ull << (loc & 63u)) - 1ull));
}

// The part of a rectangle inside bin (bx, by), clipped.
__device__ __forceinline__ TileRect clip_to_bin(const TileRect &r, const BinGrid &g, uint32_t bx,
                                                uint32_t by) {
  return TileRect{max(r.x0, bx << g.sx), max(r.y0, by << g.sy), min(r.x1, (bx + 1) << g.sx),
                  min(r.y1, (by + 1) << g.sy)};
}

// Bits of bin (bx, by) (tile (tx, ty) at bit (ty - by 2^sy) 2^sx + tx - bx 2^sx)
// of the kept tiles `keep` (row-major in r, at most kKeepBits tiles).
__device__ __forceinline__ uint32_t bin_tiles(const TileRect &r, uint64_t keep, const BinGrid &g,
                                              uint32_t bx, uint32_t by) {
  const TileRect c = clip_to_bin(r, g, bx, by);
  if (c.x0 >= c.x1) return 0u;
  const uint32_t w = r.x1 - r.x0, cw = c.x1 - c.x0;
  const uint64_t row = (1ull << cw) - 1ull;  // cw <= 2^sx <= 32
  uint32_t bits = 0;
  for (uint32_t ty = c.y0; ty < c.y1; ++ty) {
    const uint32_t b = (uint32_t)((keep >> ((ty - r.y0) * w + (c.x0 - r.x0))) & row);
    bits |= b << (((ty - (by << g.sy)) << g.sx) + (c.x0 - (bx << g.sx)));
  }
  return bits;
}

// Barrier that orders LDS only: global loads and atomics stay in flight across
// it.  (So do stores across __syncthreads, which orders them within the block.)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Exclusive scan of one value per thread over a block of NT threads; tmp:
// NT / 64 words.  Ends with a barrier (tmp may be reused at once).
template <int NT>
__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t *tmp, uint32_t *total) {
  constexpr int kW = NT / kWave;
  const int w = threadIdx.x / kWave, l = __lane_id();
  const uint32_t inc = wave_incl_scan(v);
  if (l == kWave - 1) tmp[w] = inc;
  lds_barrier();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int i = 0; i < kW; ++i) {
    const uint32_t s = tmp[i];
    if (i < w) off += s;
    tot += s;
  }
  lds_barrier();
  *total = tot;
  return off + inc - v;
}

// Two exclusive scans over a block of NT threads at once.
template <int NT>
__device__ __forceinline__ void block_scan2(uint32_t &a, uint32_t &b, uint32_t *ta, uint32_t *tb,
                                            uint32_t &total_a, uint32_t &total_b) {
  const int w = threadIdx.x / kWave, l = __lane_id();
  const uint32_t ia = wave_incl_scan(a), ib = wave_incl_scan(b);
  if (l == kWave - 1) {
    ta[w] = ia;
    tb[w] = ib;
  }
  lds_barrier();
  uint32_t oa = 0, ob = 0, sa = 0, sb = 0;
#pragma unroll
  for (int i = 0; i < NT / kWave; ++i) {
    const uint32_t va = ta[i], vb = tb[i];
    if (i < w) {
      oa += va;
      ob += vb;
    }
    sa += va;
    sb += vb;
  }
  lds_barrier();
  a = oa + ia - a;
  b = ob + ib - b;
  total_a = sa;
  total_b = sb;
}

// Block number -> item so that each XCD's blocks (b % kXcds) take consecutive
// items: neighbouring bins' data share cache lines.  Items are n; the grid is
// xcd_blocks(n), and a block whose result is >= n has no item.
__host__ __device__ inline uint32_t xcd_blocks(uint32_t n) { return (n + kXcds - 1) / kXcds * kXcds; }
__device__ __forceinline__ uint32_t xcd_item(uint32_t b, uint32_t n) {
  const uint32_t per = (n + kXcds - 1) / kXcds;
  return b % kXcds * per + b / kXcds;
}

// Entry i of a block's group from the front, large survivor i from the back.
struct GroupEntry {
  uint32_t key, slot, tiles;
};
__device__ __forceinline__ GroupEntry *group_entry(const RasterWs &ws, uint32_t block, uint32_t i) {
  return reinterpret_cast<GroupEntry *>(ws.group + (size_t)block * kGroupWords) + i;
}
__device__ __forceinline__ uint4 *group_large(const RasterWs &ws, uint32_t block, uint32_t i) {
  return reinterpret_cast<uint4 *>(ws.group + ((size_t)block + 1) * kGroupWords) - 1 - i;
}

RasterWs raster_layout(void *base, int64_t gcap, int64_t pcap, int32_t W, int32_t H);

// dst[i] = BF16 bits of src[i] rounded to nearest even, i < count (device
// arrays); enqueues one kernel on s.
hipError_t launch_round_bf16(const float *src, uint16_t *dst, int64_t count, hipStream_t s);
// The bins of each band, in depth order, into the tile lists (after the
// projection has grouped the survivors): the bin sort once per band of bin rows,
// then the scan and the lists once.
hipError_t launch_bin_sort(const RasterWs &ws, int band_row0, int rows, hipStream_t s);
hipError_t launch_tile_scan(const RasterWs &ws, bool train, hipStream_t s);
hipError_t launch_tile_lists(const RasterWs &ws, bool train, bool ordered, hipStream_t s);

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct CamParams {
  float R[9], C[3], fx, fy, cx, cy, z_near;
  int W, H;
};

constexpr uint32_t kSpinLimit = 1u << 22;  // bound of a wait on other blocks

// ---------------------------------------------------------------------------
// chained scan: decoupled look-back over one value per partition
// ---------------------------------------------------------------------------

constexpr uint32_t kLbAgg = 1u << 30;       // status flag: partition aggregate
constexpr uint32_t kLbInc = 2u << 30;       // status flag: inclusive prefix
constexpr uint32_t kLbVal = (1u << 30) - 1;  // value bits; values saturate here

__device__ __forceinline__ uint32_t sat_add(uint32_t a, uint32_t b) {
  const uint32_t s = a + b;  // a, b <= kLbVal, so no wrap
  return s > kLbVal ? kLbVal : s;
}

// Called by all 64 lanes of one wave.  Publishes partition `part`'s
// aggregate `agg` (<= kLbVal), sums the predecessors' values back to the
// nearest inclusive one, 64 partitions per round trip, publishes the
// inclusive value and returns the exclusive prefix (saturating at kLbVal).
// status[] must be zero before the first partition publishes.  A wait that
// exceeds kSpinLimit sets *err and returns what it has.
__device__ __forceinline__ uint32_t chained_lookback(uint32_t *status, uint32_t part, uint32_t agg,
                                                     uint32_t *err, uint32_t spin_limit) {
  const int l = __lane_id();
  if (l == 0) st_rel(&status[part], (part == 0 ? kLbInc : kLbAgg) | agg);
  uint32_t excl = 0;
  int64_t p = (int64_t)part - 1;
  uint32_t spins = 0;
  while (p >= 0) {
    const int64_t q = p - l;
    const uint32_t s = q >= 0 ? ld_acq(&status[q]) : kLbInc;  // before partition 0: inclusive 0
    const uint64_t ready = ballot((s & ~kLbVal) != 0u);
    const uint64_t inc = ballot((s & ~kLbVal) == kLbInc);
    const int first = inc ? __builtin_ctzll(inc) : 64;
    const uint64_t need = first < 63 ? ((2ull << first) - 1ull) : ~0ull;
    if ((ready & need) != need) {
      if (++spins > spin_limit) {
        if (l == 0) atomicOr(err, 1u);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    uint32_t v = ((need >> l) & 1ull) ? (s & kLbVal) : 0u;
    // saturating wave sum: 64 values of 30 bits fit in 36 bits
    uint64_t v64 = v;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v64 += __shfl_xor(v64, o, 64);
    excl = sat_add(excl, (uint32_t)(v64 > kLbVal ? kLbVal : v64));
    if (first < 64) break;
    p -= 64;
  }
  if (l == 0 && part > 0) st_rel(&status[part], kLbInc | sat_add(excl, agg));
  return excl;
}


// May the computed exponent of the entry exceed log2(alpha_max) at a pixel of
// the tile whose first pixel centre is (X0, Y0)?  Exactly p <= log2 op, since
// the quadratic is nowhere positive.  The conic's, the products' and the
// differences' rounding errors add up to less than 64 x 2^-24 times the sum of
// the terms' magnitudes over the tile (|dx|, |dy| reach at least 7.5, so the
// terms of d are smaller than those of p); exp2 and log2 are within 2^-16.
// Not-a-number and infinite terms count as "may".
__device__ __forceinline__ bool may_clamp(float lamax, const float4 &A, const float4 &B, float X0,
                                          float Y0) {
  const float DX = fabsf(A.x - (X0 + 7.5f)) + 7.5f, DY = fabsf(A.y - (Y0 + 7.5f)) + 7.5f;
  const float M = fabsf(A.z) * DX * DX + fabsf(A.w) * DX * DY + fabsf(B.x) * DY * DY + fabsf(B.y);
  return !(B.y + 0x1p-18f * M + 0x1p-16f < lamax);
}

}  // namespace octgs
