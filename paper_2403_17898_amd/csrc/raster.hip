// Forward rasterizer (Octree-GS Sec. III-A: EWA projection of each 3D
// Gaussian to a 2D one, tile-based front-to-back depth ordering, and the
// alpha blending of Eq. 2).
//
// Stages, all on one stream with device-resident counts (the binning kernels
// after the projection are in bins.hip):
//   project   per Gaussian slot: culls, 2D covariance, conic, 3-sigma tile
//             rectangle, depth key, the tiles that the 3-sigma ellipse meets
//             (tile_meets_ellipse); survivors grouped by screen bin
//   bin sort  per bin of up to 8 x 4 tiles, one block: collects the bin's
//             entries, sorts them by (depth, slot) in LDS, counts its tiles
//   tile scan bins of more than 4,096 entries, by all blocks; [start, end) per
//             tile
//   tile lists per bin: each tile takes its entries from the bin's ordered
//             list
//   composite one wave per 16x16 tile (four pixels of a column per lane),
//             batches of 64 Gaussians staged in LDS, exit once every pixel
//             is done; on small images eight waves per 64 pixels
//
// The (tile, depth, slot) order is that of one sort of 64-bit tile|depth keys
// over all pairs.  Sorting each bin's survivors instead (a survivor meets
// about two bins and a dozen tiles) keeps the sort inside LDS, and the pairs
// are written once, in place.  Before, the survivors were compacted and
// radix-sorted by depth (4 passes), their pairs emitted in that order and
// radix-sorted by tile (2 passes): eleven dependent kernels of 5 to 23 us,
// 138 us together on a 1080p view of 270k slots and 862k pairs; these four
// take 63 us (25, 21, 7 and 10).
//
// Decisions (culls, rectangle, depth key, tile test) use the fixed FP32
// operation sequences documented at project_decide and tile_meets_ellipse;
// continuous values are FP32.
#include "octgs_internal.h"

#include <type_traits>

namespace octgs {

namespace {

typedef CamParams Cam;

__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// Canonical FP32 projection decisions and FP32 continuous outputs for one
// Gaussian (attributes g[14]).  Sequence:
//   cull unless opacity > 0
//   d = mean - C; (xc, yc, zc) rows fmaf(R0, d0, fmaf(R1, d1, R2 * d2)); cull unless zc > z_near
//   yy=y*y zz=z*z xx=x*x xy=x*y xz=x*z yz=y*z wx=w*x wy=w*y wz=w*z
//   Rq = [1-2(yy+zz), 2(xy-wz), 2(xz+wy); 2(xy+wz), 1-2(xx+zz), 2(yz-wx); 2(xz-wy), 2(yz+wx), 1-2(xx+yy)]
//   M_ab = Rq_ab * s_b; S_ab = fmaf(M_a0, M_b0, fmaf(M_a1, M_b1, M_a2 * M_b2))
//   lx = jac_clamp * ((0.5 * W) / fx); rx = xc / zc; tx = min(lx, max(-lx, rx)) * zc (y alike)
//   zc2 = zc * zc; J00 = fx / zc; J02 = -((fx * tx) / zc2); J11 = fy / zc; J12 = -((fy * ty) / zc2)
//   T0_c = fmaf(J00, R_0c, J02 * R_2c); T1_c = fmaf(J11, R_1c, J12 * R_2c)
//   u_a = fmaf(S_a0, T0_0, fmaf(S_a1, T0_1, S_a2 * T0_2)); v_a likewise with T1
//   a = dot(T0, u) + dil; b = dot(T1, u); c = dot(T1, v) + dil;  dot = fmaf chain
//   det = a * c - b * b; cull unless det > 0
//   mid = 0.5 * (a + c); lam = mid + sqrtf(fmaxf(mid * mid - det, 0)); r = ceilf(3 * sqrtf(lam))
//   px = fmaf(fx, rx, cx); py = fmaf(fy, ry, cy)
//   x0 = clamp(floorf((px - r) * 0.0625)), x1 = clamp(floorf((px + r) * 0.0625) + 1) to [0, tiles]
//   cull if x0 >= x1 or y0 >= y1
struct ProjOut {
  float mx, my, ca, cb, cc, zc;
  int x0, y0, x1, y1;
};

__device__ __forceinline__ bool project_decide(const Cam &k, float dil, float jc, int tiles_x,
                                               int tiles_y, const float *g, ProjOut &o) {
  if (!(g[10] > 0.0f)) return false;
  const float d0 = g[0] - k.C[0], d1 = g[1] - k.C[1], d2 = g[2] - k.C[2];
  const float xc = fma_(k.R[0], d0, fma_(k.R[1], d1, k.R[2] * d2));
  const float yc = fma_(k.R[3], d0, fma_(k.R[4], d1, k.R[5] * d2));
  const float zc = fma_(k.R[6], d0, fma_(k.R[7], d1, k.R[8] * d2));
  if (!(zc > k.z_near)) return false;
  const float w = g[6], x = g[7], y = g[8], z = g[9];
  const float yy = y * y, zz = z * z, xx = x * x, xy = x * y, xz = x * z, yz = y * z;
  const float wx = w * x, wy = w * y, wz = w * z;
  float Rq[9];
  Rq[0] = 1.0f - 2.0f * (yy + zz); Rq[1] = 2.0f * (xy - wz); Rq[2] = 2.0f * (xz + wy);
  Rq[3] = 2.0f * (xy + wz); Rq[4] = 1.0f - 2.0f * (xx + zz); Rq[5] = 2.0f * (yz - wx);
  Rq[6] = 2.0f * (xz - wy); Rq[7] = 2.0f * (yz + wx); Rq[8] = 1.0f - 2.0f * (xx + yy);
  float M[9];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) M[3 * a + b] = Rq[3 * a + b] * g[3 + b];
  float S[9];
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = a; b < 3; ++b) {
      const float v = fma_(M[3 * a], M[3 * b], fma_(M[3 * a + 1], M[3 * b + 1], M[3 * a + 2] * M[3 * b + 2]));
      S[3 * a + b] = v;
      S[3 * b + a] = v;
    }
  const float lx = jc * ((0.5f * (float)k.W) / k.fx);
  const float ly = jc * ((0.5f * (float)k.H) / k.fy);
  const float rx = xc / zc, ry = yc / zc;
  const float tx = fminf(lx, fmaxf(-lx, rx)) * zc;
  const float ty = fminf(ly, fmaxf(-ly, ry)) * zc;
  const float zc2 = zc * zc;
  const float J00 = k.fx / zc, J02 = -((k.fx * tx) / zc2);
  const float J11 = k.fy / zc, J12 = -((k.fy * ty) / zc2);
  float T0[3], T1[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    T0[c] = fma_(J00, k.R[c], J02 * k.R[6 + c]);
    T1[c] = fma_(J11, k.R[3 + c], J12 * k.R[6 + c]);
  }
  float u[3], v[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    u[a] = fma_(S[3 * a], T0[0], fma_(S[3 * a + 1], T0[1], S[3 * a + 2] * T0[2]));
    v[a] = fma_(S[3 * a], T1[0], fma_(S[3 * a + 1], T1[1], S[3 * a + 2] * T1[2]));
  }
  const float ca = fma_(T0[0], u[0], fma_(T0[1], u[1], T0[2] * u[2])) + dil;
  const float cb = fma_(T1[0], u[0], fma_(T1[1], u[1], T1[2] * u[2]));
  const float cc = fma_(T1[0], v[0], fma_(T1[1], v[1], T1[2] * v[2])) + dil;
  const float det = ca * cc - cb * cb;
  if (!(det > 0.0f)) return false;
  const float mid = 0.5f * (ca + cc);
  const float lam = mid + sqrtf(fmaxf(mid * mid - det, 0.0f));
  const float r = ceilf(3.0f * sqrtf(lam));
  const float px = fma_(k.fx, rx, k.cx), py = fma_(k.fy, ry, k.cy);
  const float fx0 = floorf((px - r) * 0.0625f), fx1 = floorf((px + r) * 0.0625f) + 1.0f;
  const float fy0 = floorf((py - r) * 0.0625f), fy1 = floorf((py + r) * 0.0625f) + 1.0f;
  const float tX = (float)tiles_x, tY = (float)tiles_y;
  const int x0 = (int)fminf(fmaxf(fx0, 0.0f), tX), x1 = (int)fminf(fmaxf(fx1, 0.0f), tX);
  const int y0 = (int)fminf(fmaxf(fy0, 0.0f), tY), y1 = (int)fminf(fmaxf(fy1, 0.0f), tY);
  if (x0 >= x1 || y0 >= y1) return false;
  const float inv = 1.0f / det;
  o.mx = px; o.my = py;
  o.ca = cc * inv; o.cb = -cb * inv; o.cc = ca * inv;
  o.zc = zc;
  o.x0 = x0; o.y0 = y0; o.x1 = x1; o.y1 = y1;
  return true;
}

struct ProjArgs {
  Cam cam;
  float dil, jc;
  int tiles_x, tiles_y;
  const float *g;
  int64_t gstride;
  const uint32_t *count;
  int64_t gcap;
  RasterWs ws;
  float *gauss_w;
  int band_row0, band_rows;  // bin rows that are grouped (all of the image, but for huge images)
};

// Projection, tile tests and grouping by bin: one slot per thread, one block
// per kSlots slots.
//   - culls, 2D covariance, conic, rectangle and depth key of each slot;
//   - the tile test on every tile of the rectangles of at most kKeepBits
//     tiles: the block lays its survivors' rectangles end to end and its
//     threads take a tile each, so that neither a wave nor its lanes wait for
//     a long rectangle; the ballots are the slots' keep masks;
//   - each survivor is handed to the bins in which it keeps a tile: counted
//     per bin in LDS, then written to the block's own stretch of ws.group,
//     where the bins' entries are contiguous (ws.group_off).  A survivor over
//     more than kGroupBins bins goes to the block's large ones instead, at the
//     stretch's end, which every bin looks through.  (A block whose survivors
//     would not fit its stretch so keeps the entries of those of up to
//     kGroupBinsFull bins: 48 bytes a survivor either way at most.)
// Nothing here depends on another block, so nothing has to be cleared before
// and no global atomic is made: a bin later collects its entries from the
// blocks' stretches (a column of ws.group_off).
// Waves of 64 consecutive slots are dealt over the blocks in turn
// (slot_block): anchors lie in level order, and blocks of neighbours differed
// tenfold in the tiles that they test.
// Bound by latency and the tests' vector work: a 1080p view of 270k slots has
// 528 blocks of about 16 us (loads and projection 4, tests 6, grouping 3, the
// rest scans and writes), all resident at once: 25 us; 1.2M slots on 3840 x
// 2160 take 53, in two to three rounds.
// Block 0 clears the header and the scan's look-back words for the later
// kernels.
template <bool TRAIN>
__global__ __launch_bounds__(kSlots) void k_project(ProjArgs a) {
  constexpr int kW = kSlots / kWave;
  __shared__ float4 own[kSlots][2];
  __shared__ unsigned long long keeps[kSlots];
  __shared__ uint32_t start[kSlots + 1];
  __shared__ uint8_t mark[kW][kWave];
  extern __shared__ uint32_t hist[];  // the band's bins
  __shared__ uint32_t tmp[kW], tmp2[kW];
  __shared__ uint32_t s_vis, s_large;
  __shared__ unsigned long long s_cand;
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const RasterWs &ws = a.ws;
  const BinGrid &bg = ws.bins;
  const uint32_t n = (uint32_t)min<int64_t>(*a.count, a.gcap);
  const int nbins = a.band_rows * bg.gx;
  if (a.band_row0 == 0) {
    if (blockIdx.x == 0 && t < (int)(sizeof(RasterHeader) / 4))
      reinterpret_cast<uint32_t *>(ws.hdr)[t] = t == 0 ? n : 0u;  // n_slots is word 0
    for (int64_t i = (int64_t)blockIdx.x * kSlots + t; i < ws.scan_blocks;
         i += (int64_t)gridDim.x * kSlots)
      ws.lb_scan[i] = 0u;
  }
  const uint32_t nblk = slot_blocks(n);
  if (blockIdx.x >= nblk) return;
  const uint32_t s = ((uint32_t)w * nblk + blockIdx.x) * (uint32_t)kWave + (uint32_t)l;
  float g[kGaussFields];
  {
    const uint32_t sc = min(s, n - 1u);  // unconditional loads, all in flight together
#pragma unroll
    for (int f = 0; f < kGaussFields; ++f) g[f] = a.g[f * a.gstride + sc];
  }
  for (int i = t; i < nbins; i += kSlots) hist[i] = 0u;
  mark[w][l] = 0;
  if (t == 0) {
    s_vis = 0u;
    s_large = 0u;
    s_cand = 0ull;
  }
  ProjOut o;
  // (tile coordinates are kept in 16 bits: an image of more than 65,535 tiles
  // in one direction ends there)
  const bool vis = s < n &&
                   project_decide(a.cam, a.dil, a.jc, min(a.tiles_x, kMaxTileCoord),
                                  min(a.tiles_y, kMaxTileCoord), g, o);
  TileRect r = {0u, 0u, 0u, 0u};
  if (vis) {
    float4 *p = ws.proj + 3 * (size_t)s;
    p[0] = make_float4(o.mx, o.my, -0.5f * kLog2e * o.ca, -kLog2e * o.cb);
    p[1] = make_float4(-0.5f * kLog2e * o.cc, log2f(g[10]), g[11], g[12]);
    p[2] = make_float4(g[13], o.ca, o.cb, o.cc);
    r = TileRect{(uint32_t)o.x0, (uint32_t)o.y0, (uint32_t)o.x1, (uint32_t)o.y1};
  }
  if (a.gauss_w && s < n) a.gauss_w[s] = 0.0f;
  const uint32_t tiles = rect_tiles(r);  // 0 for a culled slot
  const bool flat = vis && tiles <= kKeepBits;
  const uint64_t vm = ballot(vis);
  if (l == 0 && s < n) ws.vis_mask[s >> 6] = vm;
  const uint32_t csum = wave_sum(tiles);  // an image has at most 2^24 tiles

  // the block's rectangles of at most kKeepBits tiles, end to end
  uint64_t keep = 0;
  {
    uint32_t ci = flat ? 1u : 0u, ex = flat ? tiles : 0u, nflat, total;
    block_scan2<kSlots>(ci, ex, tmp, tmp2, nflat, total);
    if (flat) {
      start[ci] = ex;
      keeps[ci] = 0ull;
      own[ci][0] = make_float4(o.mx, o.my, o.ca, o.cb);
      own[ci][1] = make_float4(o.cc, __uint_as_float(r.x0 | (r.y0 << 16)),
                               __uint_as_float(r.x1 - r.x0), __uint_as_float(tiles));
    }
    if (t == 0) start[nflat] = total;
    lds_barrier();
    // each wave takes consecutive stretches of 64 tiles
    const uint32_t per = ((total + kWave - 1) / kWave + kW - 1) / kW * kWave;
    const uint32_t q0 = min((uint32_t)w * per, total), q1 = min(q0 + per, total);
    uint32_t of = 0;  // owner of the stretch's first tile: the last that starts at or before it
    for (uint32_t st = kSlots / 2; st > 0; st >>= 1)
      if (of + st < nflat && start[of + st] <= q0) of += st;
    for (uint32_t b0 = q0; b0 < q1; b0 += kWave) {
      // rectangles that start in the stretch mark their first tile
      const uint32_t p = start[min(of + (uint32_t)l, nflat)] - b0;
      if (l > 0 && p < (uint32_t)kWave) mark[w][p] = 1;
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      const uint64_t sm = ballot(mark[w][l] != 0);
      __builtin_amdgcn_wave_barrier();
      mark[w][l] = 0;
      const bool in = b0 + (uint32_t)l < q1;
      const uint32_t lo = min(of + (uint32_t)__popcll(sm & (lanemask_lt() | (1ull << l))), nflat - 1u);
      of += (uint32_t)__popcll(sm);
      const float4 u = own[lo][0], v = own[lo][1];
      const uint32_t xy = __float_as_uint(v.y), wd = __float_as_uint(v.z);
      const uint32_t loc = min(b0 + (uint32_t)l, total - 1u) - start[lo];
      // row and column of the tile: a float quotient, exact after one
      // correction step (loc < 64)
      uint32_t row = (uint32_t)((float)loc * __builtin_amdgcn_rcpf((float)wd));
      const int32_t rem = (int32_t)(loc - row * wd);
      row = rem < 0 ? row - 1 : (rem >= (int32_t)wd ? row + 1 : row);
      const bool hit = in && tile_meets_ellipse(u.x, u.y, u.z, u.w, v.x,
                                                (xy & 0xffffu) + (loc - row * wd),
                                                (xy >> 16) + row, ws.xmax, ws.ymax);
      const uint64_t m = ballot(hit);
      // the owner's first lane in the wave adds its stretch of the ballot
      if (in && (l == 0 || loc == 0)) {
        const uint32_t len = min(__float_as_uint(v.w) - loc, (uint32_t)(kWave - l));
        const uint64_t bits = (m >> l) & (len < 64u ? (1ull << len) - 1ull : ~0ull);
        if (bits) atomicOr(&keeps[lo], (unsigned long long)(bits << loc));
      }
    }
    lds_barrier();
    if (flat) keep = keeps[ci];
  }
  if (vis) ws.rect[s] = make_ulonglong2(pack_rect(o.x0, o.y0, o.x1, o.y1), keep);

  // bins of this band that the survivor meets
  const uint32_t row0 = (uint32_t)a.band_row0, row1 = row0 + (uint32_t)a.band_rows;
  const uint32_t bx0 = r.x0 >> bg.sx, nbx = vis ? ((r.x1 - 1u) >> bg.sx) - bx0 + 1u : 0u;
  const uint32_t by0 = r.y0 >> bg.sy, nby = vis ? ((r.y1 - 1u) >> bg.sy) - by0 + 1u : 0u;
  const uint32_t nb = nbx * nby;
  uint32_t words, pn = TRAIN ? (flat ? (uint32_t)__popcll(keep) : tiles) : 0u, pairs;
  uint32_t want = nb <= kGroupBins ? 3u * nb : 4u;
  block_scan2<kSlots>(want, pn, tmp, tmp2, words, pairs);
  const uint32_t most = words <= kGroupWords ? kGroupBins : kGroupBinsFull;
  const bool small = vis && nb <= most;
  if (TRAIN) {
    if (vis) ws.pair_base[s] = pn;
    if (t == 0) ws.blk_pairs[blockIdx.x] = pairs;
  }
  // place among the bin's entries and tiles there, for up to kInReg bins; more
  // are rare and worked out twice
  constexpr int kInReg = 4;
  uint32_t at[kInReg], bits[kInReg], bin[kInReg];
  uint32_t meets = 0;  // more bins: bit j, the j-th of the rectangle (row-major) gets it
  const bool few = small && nb <= (uint32_t)kInReg;
  // (the tests' staging is done with)
  uint16_t (*placed)[kGroupBins] = reinterpret_cast<uint16_t (*)[kGroupBins]>(own);
  static_assert(sizeof(own) >= kSlots * kGroupBins * 2, "places fit the staging");
#pragma unroll
  for (int j = 0; j < kInReg; ++j) {
    at[j] = bits[j] = bin[j] = 0u;
    if (few && (uint32_t)j < nb) {
      const uint32_t jy = nbx == 1 ? j : (nbx == 2 ? j >> 1 : 0);  // nbx <= 4 here
      const uint32_t x = bx0 + (uint32_t)j - jy * nbx, y = by0 + jy;
      if (y >= row0 && y < row1) bits[j] = flat ? bin_tiles(r, keep, bg, x, y) : kTilesUnknown;
      if (bits[j]) {
        bin[j] = (y - row0) * (uint32_t)bg.gx + x;
        at[j] = atomicAdd(&hist[bin[j]], 1u);
      }
    }
  }
  if (small && !few) {
    uint32_t j = 0;
    for (uint32_t y = by0; y < by0 + nby; ++y)
      for (uint32_t x = bx0; x < bx0 + nbx; ++x, ++j)
        if (y >= row0 && y < row1 && (!flat || bin_tiles(r, keep, bg, x, y))) {
          meets |= 1u << j;
          placed[t][j] = (uint16_t)atomicAdd(&hist[(y - row0) * (uint32_t)bg.gx + x], 1u);
        }
  }
  const uint64_t lm = ballot(vis && !small);
  uint32_t lbase = 0;
  if (l == 0) {
    if (lm) lbase = atomicAdd(&s_large, (uint32_t)__popcll(lm));
    if (vm) atomicAdd(&s_vis, (uint32_t)__popcll(vm));
    if (csum) atomicAdd(&s_cand, (unsigned long long)csum);
  }
  lbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)lbase);
  if (vis && !small) {
    const uint64_t rc = pack_rect(o.x0, o.y0, o.x1, o.y1);
    *group_large(ws, blockIdx.x, lbase + (uint32_t)__popcll(lm & lanemask_lt())) =
        make_uint4((uint32_t)rc, (uint32_t)(rc >> 32), __float_as_uint(o.zc), s);
  }
  lds_barrier();

  // starts of the bins' entries in the block's stretch
  {
    const int per = (nbins + kSlots - 1) / kSlots;  // consecutive bins per thread
    const int i0 = min(t * per, nbins), i1 = min(i0 + per, nbins);
    uint32_t sum = 0;
    for (int i = i0; i < i1; ++i) sum += hist[i];
    uint32_t tot;
    uint32_t run = block_scan<kSlots>(sum, tmp, &tot);
    uint16_t *row = ws.group_off + (size_t)blockIdx.x * ws.group_pitch;
    for (int i = i0; i < i1; ++i) {
      const uint32_t c = hist[i];
      hist[i] = run;
      row[i] = (uint16_t)run;
      run += c;
    }
    if (t == 0) row[nbins] = (uint16_t)tot;
  }
  lds_barrier();
  GroupEntry *grp = group_entry(ws, blockIdx.x, 0u);
  const uint32_t key = __float_as_uint(o.zc);
#pragma unroll
  for (int j = 0; j < kInReg; ++j)
    if (bits[j]) grp[hist[bin[j]] + at[j]] = GroupEntry{key, s, bits[j]};
  if (meets) {
    uint32_t j = 0;
    for (uint32_t y = by0; y < by0 + nby; ++y)
      for (uint32_t x = bx0; x < bx0 + nbx; ++x, ++j)
        if ((meets >> j) & 1u)
          grp[hist[(y - row0) * (uint32_t)bg.gx + x] + placed[t][j]] =
              GroupEntry{key, s, flat ? bin_tiles(r, keep, bg, x, y) : kTilesUnknown};
  }
  if (t == 0) {
    ws.blk_vis[blockIdx.x] = s_vis;
    ws.blk_large[blockIdx.x] = s_large;
    ws.blk_cand[blockIdx.x] = (uint32_t)std::min<uint64_t>(s_cand, kLbVal);
  }
}

struct CompArgs {
  RasterWs ws;
  int W, H;
  int ordered;  // blocks take their tile from ws.tile_order
  float alpha_max, alpha_min, t_min, bg[3];
  float *rgb, *T_final;
  uint32_t *last;
  float *gauss_w;
  uint32_t *status;  // nullable: the frame's pair-overflow / look-back bits are OR-ed in
};

// One 16x16 tile per block of one wave (64 threads); each thread owns four
// vertically adjacent pixels of one column, so the Gaussian's column terms
// are shared four ways.  Batches of kFwdBatch list entries are staged in LDS.
// Per entry the exponent of the first pixel is evaluated directly and the next
// three by finite differences of the quadratic in dy (exact in real
// arithmetic; in FP32 within a few ulps of |p|):
//   dx = x - mx; dy = y0 - my
//   p0 = fma(C' dy, dy, fma(B' dx, dy, fma(A' dx, dx, log2 op)))
//   d0 = p(dy + 1) - p(dy) = fma(C', 2 dy + 1, B' dx);  d(k+1) = d(k) + 2 C'
//   p(k+1) = p(k) + d(k)
//   a = min(alpha_max, exp2(p)) = min(alpha_max, op G')
// A pixel is done once T < t_min: from then on it blends nothing.  T of a done
// pixel is kept aside and replaced by -0: w = a |T| is then +0, which leaves
// the colour and T = -0 as they are, and as an integer -0 is no smaller than
// t_min.  Entries go in groups of kGroup: the weights of all of them are
// worked out as if no pixel got done in the group; as T only falls, one
// integer minimum over the thread's pixels at the group's end and one compare
// tell if that holds, and if not the pixels of which some lane got done are
// walked again: as T falls on, the entries that leave it below t_min are the
// group's last ones, so each compare stands for itself and no chain of them
// forms.  So an entry costs no select and no compare of its own, and the alphas
// of a group do not wait for each other.  min(alpha_max, .) is left out for
// groups of entries whose exponent cannot reach log2(alpha_max) in this tile
// (may_clamp).  Where alphas may lie outside [0, 1] (t_falls) entries go one at a
// time, with a select and a compare each (step_any).
// Bound by vector issue (about 40 instructions per entry of four pixels a
// lane; 54 with the selects).  3840 x 2160, 2.3M pairs: 215 -> 187 us; 1920 x
// 1080, 0.86M: 97 -> 85; a training view of 1600 x 1066, 0.67M: 77 -> 64.  Lists
// of about 1,000 entries in 725 tiles, in most groups of which some pixel gets
// done (300k Gaussians within 400 x 400 px): 244 with a select per entry, 283
// where the walk kept a chain of done flags for all four pixels, 242 now.
// Groups of 2, 4, 8 and 16 take 100, 92, 87 and 93 us at 1920 x 1080.  Four
// waves per SIMD (117 registers): held to five the walk's values spill.
constexpr int kFwdThreads = 64;
constexpr int kFwdBatch = 64;     // list entries staged in LDS per batch, one per lane
constexpr int kPx = 4;            // pixels of a column
constexpr int kGroup = 8;         // entries per check for done pixels

template <bool LOG>
struct CompLds {
  float4 sA[kFwdBatch], sB[kFwdBatch], sC[kFwdBatch];  // (mx, my, A', B') (C', log2 op, 2 C', -) (r, g, b, -)
  uint32_t s_slot[LOG ? kFwdBatch : 1];
  float s_w[LOG ? kFwdBatch : 1];
};

// The conditions of the earlier stages are final in the composite: one thread
// adds them to the caller's status word.
__device__ __forceinline__ void add_status(const CompArgs &a) {
  if (a.status && blockIdx.x == 0 && threadIdx.x == 0) {
    const uint32_t f = (a.ws.hdr->pair_overflow ? OCTGS_STATUS_PAIR_OVERFLOW : 0u) |
                       (a.ws.hdr->sync_error ? OCTGS_STATUS_SYNC_ERROR : 0u);
    if (f) atomicOr(a.status, f);
  }
}

// T only falls and stays in [0, 1], as alphas lie in [0, 1].
__host__ __device__ __forceinline__ bool t_falls(const CompArgs &a) {
  return a.alpha_max >= 0.0f && a.alpha_max <= 1.0f;
}

// Where t_falls: T as an integer below this has crossed t_min.
__device__ __forceinline__ uint32_t t_bits(const CompArgs &a) {
  return a.t_min > 0.0f ? __float_as_uint(a.t_min) : 0u;
}

// The LDS lives in the kernel and is passed in, so the instantiations share
// one allocation.
template <bool LOG, bool AMIN, bool LAST>
__device__ __forceinline__ void composite_tile(const CompArgs &a, CompLds<LOG> &lds) {
  float4 *sA = lds.sA, *sB = lds.sB, *sC = lds.sC;
  uint32_t *s_slot = lds.s_slot;
  float *s_w = lds.s_w;
  const int32_t tile = a.ordered ? (int32_t)a.ws.tile_order[blockIdx.x]
                                 : tile_of_block(blockIdx.x, a.ws.tiles_x, a.ws.tiles_y);
  if (tile < 0) return;
  const int tx = tile % a.ws.tiles_x, ty = tile / a.ws.tiles_x;
  const int t = threadIdx.x;
  const int px = tx * kTile + (t % kTile), py0 = ty * kTile + kPx * (t / kTile);
  const float fx = (float)px + 0.5f, fy = (float)py0 + 0.5f;
  const uint32_t start = __builtin_amdgcn_readfirstlane(a.ws.ranges[2 * tile]);
  const uint32_t end = __builtin_amdgcn_readfirstlane(a.ws.ranges[2 * tile + 1]);
  const uint32_t *vals = a.ws.tval;
  const float4 *proj = a.ws.proj;
  const float amax = a.alpha_max, amin = a.alpha_min, tmin = a.t_min;
  const uint32_t tbits = t_bits(a);
  const bool falling = t_falls(a);
  const float lamax = log2f(amax);
  float T[kPx], Tdone[kPx], cr[kPx], cg[kPx], cb[kPx];
  uint32_t last[kPx];
  uint32_t done = 0;  // bit k: pixel k
#pragma unroll
  for (int k = 0; k < kPx; ++k) {
    const bool in = px < a.W && py0 + k < a.H;
    T[k] = in ? 1.0f : -0.0f;
    done |= in ? 0u : 1u << k;
    Tdone[k] = 0.0f;
    cr[k] = 0.0f; cg[k] = 0.0f; cb[k] = 0.0f;
    last[k] = end - start;
  }
  const uint32_t outside = done;
  constexpr uint32_t kAll = (1u << kPx) - 1u;
  for (uint32_t b0 = start; b0 < end; b0 += kFwdBatch) {
    // one wave: the barrier only orders LDS reuse across batches
    __syncthreads();
    uint64_t clamp;  // bit j: entry j may need min(alpha_max, .)
    {
      const uint32_t s = vals[min(b0 + t, end - 1u)];
      if (LOG) s_slot[t] = s;
      const float4 A = proj[3 * (size_t)s], B = proj[3 * (size_t)s + 1];
      sA[t] = A;
      sB[t] = make_float4(B.x, B.y, B.x + B.x, 0.0f);
      sC[t] = make_float4(B.z, B.w, proj[3 * (size_t)s + 2].x, 0.0f);
      clamp = ballot(may_clamp(lamax, A, B, (float)(tx * kTile) + 0.5f, (float)(ty * kTile) + 0.5f));
    }
    __syncthreads();
    const int nb = __builtin_amdgcn_readfirstlane((int)min((uint32_t)kFwdBatch, end - b0));
    const uint32_t base = b0 - start + 1u;
    // returns true once every pixel is done
    auto step = [&](int j, auto ngroup, auto clamped) -> bool {
      constexpr int G = decltype(ngroup)::value;
      constexpr bool CLAMP = decltype(clamped)::value;
      float w[G][kPx], T0[kPx];
#pragma unroll
      for (int k = 0; k < kPx; ++k) T0[k] = T[k];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float4 A = sA[j + g];
        const float4 B = sB[j + g];
        const float dx = fx - A.x;
        const float adx = fma_(A.z * dx, dx, B.y);
        const float bdx = A.w * dx;
        const float dy = fy - A.y;
        float p = fma_(B.x * dy, dy, fma_(bdx, dy, adx));
        float d = fma_(B.x, fma_(2.0f, dy, 1.0f), bdx);
#pragma unroll
        for (int k = 0; k < kPx; ++k) {
          if (k > 0) {
            p += d;
            d += B.z;
          }
          float al = __builtin_amdgcn_exp2f(p);
          if (CLAMP) al = fminf(amax, al);
          if (AMIN) al = al < amin ? 0.0f : al;
          w[g][k] = al * fabsf(T[k]);
          T[k] = T[k] - w[g][k];
        }
      }
      uint32_t low = ~0u;
#pragma unroll
      for (int k = 0; k < kPx; ++k) low = min(low, __float_as_uint(T[k]));
      bool stop = false;
      if (ballot(low < tbits) != 0ull) {
        // as T only falls, the entries that a pixel counts are those before the
        // first that leaves it below t_min, and that one; `last` is that
        // entry, else the list length
#pragma unroll
        for (int k = 0; k < kPx; ++k) {
          if (ballot(__float_as_uint(T[k]) < tbits) == 0ull) continue;
          float Tg = T0[k], Te = T0[k];  // as if no pixel got done; left at
          bool under = false;            // false where done (T0 = -0, w = 0)
          uint32_t left = 0;
#pragma unroll
          for (int g = 0; g < G; ++g) {
            Tg -= w[g][k];
            Te = under ? Te : Tg;
            w[g][k] = under ? 0.0f : w[g][k];
            under = __float_as_uint(Tg) < tbits;
            if (LAST) left += under ? 1u : 0u;
          }
          if (LAST) last[k] = under ? base + (uint32_t)(j + G) - left : last[k];
          Tdone[k] = under ? Te : Tdone[k];
          T[k] = under ? -0.0f : T[k];
          done |= under ? 1u << k : 0u;
        }
        stop = __all(done == kAll);
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const float4 C = sC[j + g];
        float wsum = 0.0f;
#pragma unroll
        for (int k = 0; k < kPx; ++k) {
          cr[k] = fma_(w[g][k], C.x, cr[k]);
          cg[k] = fma_(w[g][k], C.y, cg[k]);
          cb[k] = fma_(w[g][k], C.z, cb[k]);
          if (LOG) wsum += w[g][k];
        }
        if (LOG) {
          const float ws = wave_sum_f(wsum);
          if (__lane_id() == 0) s_w[j + g] = ws;
        }
      }
      return stop;
    };
    // one entry, any alpha_max and t_min: T may be negative and rise again
    auto step_any = [&](int j) -> bool {
      const float4 A = sA[j], B = sB[j], C = sC[j];
      const float dx = fx - A.x;
      const float adx = fma_(A.z * dx, dx, B.y);
      const float bdx = A.w * dx;
      const float dy = fy - A.y;
      float p = fma_(B.x * dy, dy, fma_(bdx, dy, adx));
      float d = fma_(B.x, fma_(2.0f, dy, 1.0f), bdx);
      float wsum = 0.0f;
#pragma unroll
      for (int k = 0; k < kPx; ++k) {
        if (k > 0) {
          p += d;
          d += B.z;
        }
        float al = fminf(amax, __builtin_amdgcn_exp2f(p));
        if (AMIN) al = al < amin ? 0.0f : al;
        const bool live = !(done & (1u << k));
        const float w = live ? al * T[k] : 0.0f;
        T[k] -= w;
        cr[k] = fma_(w, C.x, cr[k]);
        cg[k] = fma_(w, C.y, cg[k]);
        cb[k] = fma_(w, C.z, cb[k]);
        if (LOG) wsum += w;
        if (live && T[k] < tmin) {
          if (LAST) last[k] = base + (uint32_t)j;
          Tdone[k] = T[k];
          done |= 1u << k;
        }
      }
      if (LOG) {
        const float ws = wave_sum_f(wsum);
        if (__lane_id() == 0) s_w[j] = ws;
      }
      return __all(done == kAll);
    };
    typedef std::integral_constant<int, kGroup> Group;
    typedef std::integral_constant<int, 1> One;
    int j = 0;
    bool stop = false;
    if (!falling)
      for (; j < nb && (LOG || !stop); ++j) stop = step_any(j);
    for (; j + kGroup <= nb && (LOG || !stop); j += kGroup)
      stop = (uint32_t)(clamp >> j) & ((1u << kGroup) - 1u)
                 ? step(j, Group(), std::true_type())
                 : step(j, Group(), std::false_type());
    for (; j < nb && (LOG || !stop); ++j) stop = step(j, One(), std::true_type());
    if (LOG) {
      __syncthreads();
      if (t < nb && s_w[t] != 0.0f) atomicAdd(&a.gauss_w[s_slot[t]], s_w[t]);
    }
    if (__all(done == kAll)) break;
  }
  const size_t plane = (size_t)a.W * a.H;
#pragma unroll
  for (int k = 0; k < kPx; ++k) {
    if (!(outside & (1u << k))) {
      const size_t pix = (size_t)(py0 + k) * a.W + px;
      const float Tk = done & (1u << k) ? Tdone[k] : T[k];
      a.rgb[pix] = fma_(Tk, a.bg[0], cr[k]);
      a.rgb[plane + pix] = fma_(Tk, a.bg[1], cg[k]);
      a.rgb[2 * plane + pix] = fma_(Tk, a.bg[2], cb[k]);
      a.T_final[pix] = Tk;
      if (LAST) a.last[pix] = last[k];
    }
  }
}

// Few tiles (kFewTiles): one wave per tile leaves most of the chip idle and the
// longest list sets the time, 0.13 us per entry.  Here a block of eight waves
// composites 64 pixels, the K-th (K = 0 .. 3) of every column of four: waves
// 3 to 7 work out the alphas of a batch, every fifth entry each, into LDS,
// while waves 0 to 2 blend the batch before it, a colour channel each (T in all
// three), which leaves three instructions per entry in the chain.  The last two
// waves also stage the batches that follow.  The operations on a pixel are those of
// composite_tile, in the same order.
// A 128 x 128 view whose longest list has 606 entries: 81 -> 19 us.  (16 waves
// a block, two of them staging only: 17 there, but half as fast again from 256
// tiles on.)  It costs 2.5 times the vector work of one wave per tile, so it
// stops paying where the chip is full: whole passes of one view with one wave
// per tile / these blocks, at 64 tiles 75 / 53 us, 256: 76 / 64, 475: 79 / 77
// (94 / 85 with longer lists), 768: 80 / 86, 1024: 80 / 96; four views in
// flight, at 64 tiles 293 / 237, 192: 294 / 265, 300: 345 / 318.
constexpr int kFewThreads = 512, kFewWaves = kFewThreads / kWave;
constexpr int kFewBlend = 3, kFewAlpha = kFewWaves - kFewBlend, kFewStage = 2;
constexpr int kFewTiles = 400;
constexpr int kRing = 4;  // staged batches: blended last, being blended, next, after next

template <bool LOG>
struct FewLds {
  float4 sA[kRing][kFwdBatch], sB[kRing][kFwdBatch];
  alignas(16) float sC[kFewBlend][kRing][kFwdBatch];
  uint32_t s_slot[kRing][kFwdBatch];
  float al[2][kFwdBatch][kWave];                      // alphas of a batch
  float wt[LOG ? 2 : 1][LOG ? kFwdBatch : 1][kWave];  // its weights
  uint32_t stop[2];
};

template <bool LOG, bool AMIN, int K>
__device__ __forceinline__ void few_alphas(const CompArgs &a, FewLds<LOG> &lds, uint32_t b, int w, int l,
                                           int nb, float fx, float fy) {
  // several entries at a time, as one alone is a chain of latencies
  constexpr int kN = 4;
  for (int j0 = w - kFewBlend; j0 < nb; j0 += kN * kFewAlpha) {
    float4 A[kN], B[kN];
#pragma unroll
    for (int u = 0; u < kN; ++u) {
      const int j = min(j0 + u * kFewAlpha, kFwdBatch - 1);
      A[u] = lds.sA[b % kRing][j];
      B[u] = lds.sB[b % kRing][j];
    }
    float al[kN];
#pragma unroll
    for (int u = 0; u < kN; ++u) {
      const float dx = fx - A[u].x;
      const float adx = fma_(A[u].z * dx, dx, B[u].y);
      const float bdx = A[u].w * dx;
      const float dy = fy - A[u].y;
      float p = fma_(B[u].x * dy, dy, fma_(bdx, dy, adx));
      float d = fma_(B[u].x, fma_(2.0f, dy, 1.0f), bdx);
#pragma unroll
      for (int k = 0; k < K; ++k) {
        p += d;
        d += B[u].z;
      }
      al[u] = fminf(a.alpha_max, __builtin_amdgcn_exp2f(p));
      if (AMIN) al[u] = al[u] < a.alpha_min ? 0.0f : al[u];
    }
#pragma unroll
    for (int u = 0; u < kN; ++u) {
      const int j = j0 + u * kFewAlpha;
      if (j < kFwdBatch) lds.al[b & 1][j][l] = j < nb ? al[u] : 0.0f;
    }
  }
  // (the blending reads whole groups)
  for (int j = nb + w - kFewBlend; j < min((nb + kGroup - 1) / kGroup * kGroup, kFwdBatch); j += kFewAlpha)
    lds.al[b & 1][j][l] = 0.0f;
}

// ANY: for alphas outside [0, 1] (t_falls), where T may be negative and rise
// again; the blending waves then go entry by entry.
template <bool LOG, bool ANY>
__global__ __launch_bounds__(kFewThreads) void k_composite_few(CompArgs a) {
  __shared__ FewLds<LOG> lds;
  add_status(a);
  const int K = (int)(blockIdx.x % kPx);
  const uint32_t block = blockIdx.x / kPx;
  const int32_t tile = a.ordered ? (int32_t)a.ws.tile_order[block]
                                 : tile_of_block(block, a.ws.tiles_x, a.ws.tiles_y);
  if (tile < 0) return;
  const int tx = tile % a.ws.tiles_x, ty = tile / a.ws.tiles_x;
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), l = __lane_id();
  const int px = tx * kTile + (l % kTile), row0 = ty * kTile + kPx * (l / kTile), py = row0 + K;
  const float fx = (float)px + 0.5f, fy = (float)row0 + 0.5f;
  const uint32_t start = __builtin_amdgcn_readfirstlane(a.ws.ranges[2 * tile]);
  const uint32_t end = __builtin_amdgcn_readfirstlane(a.ws.ranges[2 * tile + 1]);
  const int len = (int)(end - start), nbatch = (len + kFwdBatch - 1) / kFwdBatch;
  const float tmin = a.t_min;
  const uint32_t tbits = t_bits(a);
  const bool in = px < a.W && py < a.H;
  float T = in ? 1.0f : -0.0f, Tdone = 0.0f, col = 0.0f;
  uint32_t last = (uint32_t)len;
  bool done = !in;

  // entry l of batch b: its slot (past the list's end, the last entry's), then
  // its data (there, a colour of 0)
  float4 A, B, C;
  uint32_t s = 0, s_next = 0;
  auto slot_of = [&](int b) { return a.ws.tval[start + (uint32_t)min(b * kFwdBatch + l, len - 1)]; };
  auto load = [&](int b) {
    A = a.ws.proj[3 * (size_t)s];
    B = a.ws.proj[3 * (size_t)s + 1];
    C = make_float4(B.z, B.w, a.ws.proj[3 * (size_t)s + 2].x, 0.0f);
    if (b * kFwdBatch + l >= len) C = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  };
  auto put = [&](int b) {
    lds.sA[b % kRing][l] = A;
    lds.sB[b % kRing][l] = make_float4(B.x, B.y, B.x + B.x, 0.0f);
    lds.sC[0][b % kRing][l] = C.x;
    lds.sC[1][b % kRing][l] = C.y;
    lds.sC[2][b % kRing][l] = C.z;
    lds.s_slot[b % kRing][l] = s;
  };
  // sums of batch b's weights, by the waves that wrote its alphas
  auto log_weights = [&](int b) {
    const int nb = min(kFwdBatch, len - b * kFwdBatch);
    for (int j = w - kFewBlend; j < nb; j += kFewAlpha) {
      const float ws = wave_sum_f(lds.wt[b & 1][j][l]);
      if (l == 0 && ws != 0.0f) atomicAdd(&a.gauss_w[lds.s_slot[b % kRing][j]], ws);
    }
  };
  // the last two waves stage the even and the odd batches: a batch's slots are
  // read two batches before its entries' data, and that two batches before it is
  // put down, as either takes longer to arrive than a batch to blend
  const int stage = w - (kFewWaves - kFewStage);  // 0 or 1: this wave's batches
  if (stage >= 0 && stage < nbatch) {
    s = slot_of(stage);
    s_next = slot_of(stage + 2);
    load(stage);
    put(stage);
    s = s_next;
    s_next = slot_of(stage + 4);
    load(stage + 2);
  }
  __syncthreads();
  int b = -1;
  for (; b < nbatch; ++b) {
    if (b >= 0 && (b & 1) == stage && b + 2 < nbatch) {
      put(b + 2);
      s = s_next;
      s_next = slot_of(b + 6);
      load(b + 4);
    }
    if (w < kFewBlend) {
      if (b >= 0) {
        const int nb = min(kFwdBatch, len - b * kFwdBatch);
        const float *sC = lds.sC[w][b % kRing];
        const float (*al)[kWave] = lds.al[b & 1];
        float an[kGroup], cn[kGroup];  // the next group's, read ahead
        auto read = [&](int j) {
#pragma unroll
          for (int g = 0; g < kGroup; ++g) an[g] = al[j + g][l];
#pragma unroll
          for (int g = 0; g < kGroup; g += 4) {
            const float4 v = *reinterpret_cast<const float4 *>(sC + j + g);
            cn[g] = v.x; cn[g + 1] = v.y; cn[g + 2] = v.z; cn[g + 3] = v.w;
          }
        };
        read(0);
        for (int j = 0; j < nb; j += kGroup) {
          float wt[kGroup], c[kGroup], T0 = T;
#pragma unroll
          for (int g = 0; g < kGroup; ++g) {
            wt[g] = an[g];
            c[g] = cn[g];
          }
          read(min(j + kGroup, kFwdBatch - kGroup));
#pragma unroll
          for (int g = 0; g < kGroup; ++g) {
            wt[g] = wt[g] * fabsf(T);
            T -= wt[g];
          }
          if (ANY || ballot(__float_as_uint(T) < tbits) != 0ull) {
            bool live = !done;
            float Tk = T0;
#pragma unroll
            for (int g = 0; g < kGroup; ++g) {
              if (ANY) wt[g] = al[j + g][l] * Tk;
              wt[g] = live ? wt[g] : 0.0f;
              Tk -= wt[g];
              const bool now = live && Tk < tmin;
              last = now ? (uint32_t)(b * kFwdBatch + j + g + 1) : last;
              live = live && !now;
            }
            Tdone = live || done ? Tdone : Tk;
            T = live ? Tk : -0.0f;
            done = !live;
          }
#pragma unroll
          for (int g = 0; g < kGroup; ++g) {
            col = fma_(wt[g], c[g], col);
            if (LOG && w == 0) lds.wt[b & 1][j + g][l] = wt[g];
          }
        }
        const bool all = __all(done);  // over the whole wave
        if (w == 0 && l == 0) lds.stop[b & 1] = all ? 1u : 0u;
      }
    } else {
      if (LOG && b > 0) log_weights(b - 1);
      if (b + 1 < nbatch) {
        const int nb = min(kFwdBatch, len - (b + 1) * kFwdBatch);
        const bool amin = a.alpha_min > 0.0f;
#define OCTGS_FEW_ALPHAS(KK)                                                \
  case KK:                                                                  \
    if (amin)                                                               \
      few_alphas<LOG, true, KK>(a, lds, (uint32_t)(b + 1), w, l, nb, fx, fy);    \
    else                                                                    \
      few_alphas<LOG, false, KK>(a, lds, (uint32_t)(b + 1), w, l, nb, fx, fy);   \
    break;
        switch (K) {
          OCTGS_FEW_ALPHAS(0)
          OCTGS_FEW_ALPHAS(1)
          OCTGS_FEW_ALPHAS(2)
          OCTGS_FEW_ALPHAS(3)
        }
#undef OCTGS_FEW_ALPHAS
      }
    }
    lds_barrier();
    // (a word is written again two barriers later)
    if (b >= 0 && lds.stop[b & 1]) break;
  }
  if (LOG && nbatch > 0 && w >= kFewBlend) log_weights(min(b, nbatch - 1));
  if (w >= kFewBlend || !in) return;
  const size_t plane = (size_t)a.W * a.H, pix = (size_t)py * a.W + px;
  const float Tk = done ? Tdone : T;
  a.rgb[w * plane + pix] = fma_(Tk, w == 0 ? a.bg[0] : (w == 1 ? a.bg[1] : a.bg[2]), col);
  if (w > 0) return;
  a.T_final[pix] = Tk;
  if (a.last) a.last[pix] = last;
}

template <bool LOG>
__global__ __launch_bounds__(kFwdThreads, LOG ? 1 : 4) void k_composite(CompArgs a) {
  __shared__ CompLds<LOG> lds;
  add_status(a);
  // a render that no backward follows may leave out the per-pixel entry count
  if (a.alpha_min > 0.0f) {
    if (a.last)
      composite_tile<LOG, true, true>(a, lds);
    else
      composite_tile<LOG, true, false>(a, lds);
  } else {
    if (a.last)
      composite_tile<LOG, false, true>(a, lds);
    else
      composite_tile<LOG, false, false>(a, lds);
  }
}

// The bins of an image: as large as leaves at least kWantBins of them, so that
// a small image's lists are spread over the chip too, but no larger than 8 x 4
// tiles (a mask word).  1920 x 1080: 15 x 17 bins of 8 x 4.
// Fewer, larger bins win while that many are left, as a survivor meets fewer of
// them: with at least 400 (4 x 4 there) a 1920 x 1080 view takes 148 us instead
// of 141, four in flight 755 instead of 707.
constexpr int kWantBins = 160;

BinGrid bin_grid(int tiles_x, int tiles_y) {
  BinGrid g;
  static const int shape[][2] = {{3, 2}, {2, 2}, {2, 1}, {1, 1}, {1, 0}, {0, 0}};
  for (const auto &s : shape) {
    g.sx = s[0];
    g.sy = s[1];
    g.nx = (tiles_x + (1 << g.sx) - 1) >> g.sx;
    g.ny = (tiles_y + (1 << g.sy) - 1) >> g.sy;
    if ((int64_t)g.nx * g.ny >= kWantBins) break;
  }
  // (images this wide have bins of 8 x 4 tiles, so gx <= kMaxBandBins)
  g.gx = std::min(g.nx, (kMaxTileCoord + (1 << g.sx) - 1) >> g.sx);
  g.band_rows = std::min(g.ny, std::max(1, kMaxBandBins / g.gx));
  return g;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

RasterWs raster_layout(void *base, int64_t gcap, int64_t pcap, int32_t W, int32_t H) {
  RasterWs ws;
  char *p = (char *)base;
  size_t off = 0;
  auto take = [&](size_t bytes) -> void * {
    void *r = p ? (void *)(p + off) : nullptr;
    off += align256(bytes);
    return r;
  };
  const int64_t g = std::max<int64_t>(gcap, 1), pc = std::max<int64_t>(pcap, 1);
  ws.gcap = g;
  ws.pcap = pc;
  ws.xmax = (float)W - 0.5f;
  ws.ymax = (float)H - 0.5f;
  ws.tiles_x = (W + kTile - 1) / kTile;
  ws.tiles_y = (H + kTile - 1) / kTile;
  ws.nblk_g = (int)((g + kSlots - 1) / kSlots);
  ws.bins = bin_grid(ws.tiles_x, ws.tiles_y);
  const int64_t ntiles = (int64_t)ws.tiles_x * ws.tiles_y;
  const int64_t nbins = (int64_t)ws.bins.nx * ws.bins.ny;
  ws.group_pitch = (int)((std::min<int64_t>(nbins, (int64_t)ws.bins.band_rows * ws.bins.gx) + 2) & ~1);
  ws.scan_blocks = (int)((ntiles + kScanTiles * kScanThreads - 1) / (kScanTiles * kScanThreads));
  ws.hdr = (RasterHeader *)take(sizeof(RasterHeader));
  ws.vis_mask = (uint64_t *)take((size_t)ws.nblk_g * (kSlots / kWave) * 8);
  ws.blk_vis = (uint32_t *)take((size_t)ws.nblk_g * 4);
  ws.blk_cand = (uint32_t *)take((size_t)ws.nblk_g * 4);
  ws.blk_large = (uint32_t *)take((size_t)ws.nblk_g * 4);
  ws.blk_pairs = (uint32_t *)take((size_t)ws.nblk_g * 4);
  ws.proj = (float4 *)take((size_t)kProjVec * g * 16);
  ws.rect = (ulonglong2 *)take((size_t)g * 16);
  ws.pair_base = (uint32_t *)take((size_t)g * 4);
  ws.group_off = (uint16_t *)take((size_t)ws.nblk_g * ws.group_pitch * 2);
  ws.bin_range = (uint2 *)take((size_t)nbins * 8);
  for (int i = 0; i < 2; ++i) ws.bin_slot[i] = (uint32_t *)take((size_t)pc * 4);
  for (int i = 0; i < 2; ++i) ws.bin_mask[i] = (uint32_t *)take((size_t)pc * 4);
  ws.over_bin = (uint32_t *)take((size_t)(pc / kBinCap + 1) * 8);
  // a long bin has more than kBinCap entries, so at most one slice more than
  // its share of pc / kSliceEntries
  ws.slices = (uint32_t *)take((size_t)(pc / kSliceEntries + pc / kBinCap + 1) * kSliceRow * 4);
  ws.lb_scan = (uint32_t *)take((size_t)ws.scan_blocks * 4);
  ws.tkey = (uint32_t *)take((size_t)pc * 4);
  ws.tval = (uint32_t *)take((size_t)pc * 4);
  ws.ranges = (uint32_t *)take((size_t)ntiles * 8);
  // the scan reads the counts before the lists' kernel writes the order
  ws.tile_order = (uint32_t *)take(
      4 * std::max<size_t>(tile_grid_blocks(ws.tiles_x, ws.tiles_y),
                           (size_t)ws.scan_blocks * kScanTiles * kScanThreads));
  ws.tile_count = ws.tile_order;
  // the groups are read by the bin sort and the scan, before anything writes the
  // backward's arrays (the tile lists clear rows of gpair): one place for both
  const size_t shared = off;
  ws.group = (uint32_t *)take((size_t)ws.nblk_g * kGroupWords * 4);
  const size_t fwd_end = off;
  off = shared;
  ws.dproj = (float *)take((size_t)g * 9 * 4);
  ws.gpair = (float *)take((size_t)pc * kPairRow * 4);
  ws.chunk_part = (float *)take((size_t)((pc + 63) / 64) * 18 * 4);
  off = std::max(off, fwd_end);
  ws.bytes = off;
  return ws;
}

}  // namespace octgs

using namespace octgs;

extern "C" {

size_t octgs_raster_workspace_bytes(int64_t gauss_capacity, int64_t pair_capacity, int32_t width,
                                    int32_t height) {
  if (gauss_capacity < 0 || pair_capacity < 0 || !image_tiles_ok(width, height)) return 0;
  return raster_layout(nullptr, gauss_capacity, pair_capacity, width, height).bytes;
}

int octgs_rasterize_fwd(const octgs_gaussians *g, const octgs_camera *cam,
                        const octgs_raster_params *p, int64_t pair_capacity, float *rgb,
                        float *T_final, uint32_t *last, float *gauss_w, void *wsp,
                        size_t ws_bytes, void *const *stage_events, octgs_stream stream) {
  if (!g || !cam || !p || !rgb || !T_final || !wsp) return OCTGS_EINVAL;
  if (!g->data || !g->count || g->capacity < 0 || g->capacity >= (int64_t(1) << 31))
    return OCTGS_EINVAL;
  // candidate counts saturate at 2^30 - 1, which must exceed the capacity
  if (pair_capacity < 0 || pair_capacity >= (int64_t(1) << 30) - 1) return OCTGS_EINVAL;
  if (!image_tiles_ok(cam->width, cam->height)) return OCTGS_EINVAL;
  if (!(cam->fx > 0.0f) || !(cam->fy > 0.0f)) return OCTGS_EINVAL;
  // z_near > 0 keeps every listed depth positive (the depth keys are float bits)
  if (!(cam->z_near > 0.0f)) return OCTGS_EINVAL;
  if (!(p->dilation >= 0.0f) || !(p->jac_clamp > 0.0f)) return OCTGS_EINVAL;
  if (ws_bytes < octgs_raster_workspace_bytes(g->capacity, pair_capacity, cam->width, cam->height))
    return OCTGS_ENOSPC;
  hipStream_t s = (hipStream_t)stream;
  RasterWs ws = raster_layout(wsp, g->capacity, pair_capacity, cam->width, cam->height);
  auto mark = [&](int i) {
    if (stage_events && stage_events[i]) (void)hipEventRecord((hipEvent_t)stage_events[i], s);  // timing only
  };
  ProjArgs pa;
  for (int i = 0; i < 9; ++i) pa.cam.R[i] = cam->R[i];
  for (int i = 0; i < 3; ++i) pa.cam.C[i] = cam->C[i];
  pa.cam.fx = cam->fx; pa.cam.fy = cam->fy; pa.cam.cx = cam->cx; pa.cam.cy = cam->cy;
  pa.cam.z_near = cam->z_near; pa.cam.W = cam->width; pa.cam.H = cam->height;
  pa.dil = p->dilation;
  pa.jc = p->jac_clamp;
  pa.tiles_x = ws.tiles_x;
  pa.tiles_y = ws.tiles_y;
  pa.g = g->data;
  pa.gstride = g->capacity;
  pa.count = g->count;
  pa.gcap = g->capacity;
  pa.ws = ws;
  pa.gauss_w = gauss_w;
  const bool train = (p->flags & OCTGS_RASTER_TRAIN) != 0;
  const bool ordered = (p->flags & OCTGS_RASTER_TILE_ORDER) != 0;
  // one pass over all bins, but for images of more than kMaxBandBins bins
  mark(0);
  hipError_t e = hipSuccess;
  for (int row0 = 0; row0 < ws.bins.ny && e == hipSuccess; row0 += ws.bins.band_rows) {
    pa.band_row0 = row0;
    pa.band_rows = std::min(ws.bins.band_rows, ws.bins.ny - row0);
    const size_t lds = (size_t)pa.band_rows * ws.bins.gx * sizeof(uint32_t);
    if (train)
      hipLaunchKernelGGL(k_project<true>, dim3(ws.nblk_g), dim3(kSlots), lds, s, pa);
    else
      hipLaunchKernelGGL(k_project<false>, dim3(ws.nblk_g), dim3(kSlots), lds, s, pa);
    if (row0 == 0) {
      mark(1);
      mark(2);
    }
    e = launch_bin_sort(ws, row0, pa.band_rows, s);
  }
  mark(3);
  mark(4);
  if (e == hipSuccess) e = launch_tile_scan(ws, train, s);
  mark(5);
  mark(6);
  if (e == hipSuccess) e = launch_tile_lists(ws, train, ordered, s);
  mark(7);
  if (e != hipSuccess) return OCTGS_EHIP;
  CompArgs ca;
  ca.ws = ws;
  ca.ordered = ordered ? 1 : 0;
  ca.W = cam->width;
  ca.H = cam->height;
  ca.alpha_max = p->alpha_max;
  ca.alpha_min = p->alpha_min;
  ca.t_min = p->t_min;
  for (int i = 0; i < 3; ++i) ca.bg[i] = p->bg[i];
  ca.rgb = rgb;
  ca.T_final = T_final;
  ca.last = last;
  ca.gauss_w = gauss_w;
  ca.status = g->status;
  mark(8);
  const uint32_t blocks = tile_grid_blocks(ws.tiles_x, ws.tiles_y);
  if ((int64_t)ws.tiles_x * ws.tiles_y <= kFewTiles) {
    const auto few = t_falls(ca) ? (gauss_w ? k_composite_few<true, false> : k_composite_few<false, false>)
                                 : (gauss_w ? k_composite_few<true, true> : k_composite_few<false, true>);
    hipLaunchKernelGGL(few, dim3(kPx * blocks), dim3(kFewThreads), 0, s, ca);
  } else {
    if (gauss_w)
      hipLaunchKernelGGL(k_composite<true>, dim3(blocks), dim3(kFwdThreads), 0, s, ca);
    else
      hipLaunchKernelGGL(k_composite<false>, dim3(blocks), dim3(kFwdThreads), 0, s, ca);
  }
  mark(9);
  return hipGetLastError() == hipSuccess ? OCTGS_OK : OCTGS_EHIP;
}

int octgs_raster_views(const void *wsp, int64_t gauss_capacity, int64_t pair_capacity,
                       int32_t width, int32_t height, const octgs_raster_stats **stats,
                       const uint32_t **pair_tile, const uint32_t **pair_slot,
                       const uint32_t **tile_ranges) {
  if (!wsp || width <= 0 || height <= 0 || gauss_capacity < 0 || pair_capacity < 0)
    return OCTGS_EINVAL;
  RasterWs ws = raster_layout(const_cast<void *>(wsp), gauss_capacity, pair_capacity, width, height);
  if (stats) *stats = (const octgs_raster_stats *)ws.hdr;
  if (pair_tile) *pair_tile = ws.tkey;
  if (pair_slot) *pair_slot = ws.tval;
  if (tile_ranges) *tile_ranges = ws.ranges;
  return OCTGS_OK;
}

const char *octgs_strerror(int status) {
  switch (status) {
    case OCTGS_OK: return "ok";
    case OCTGS_EINVAL: return "invalid argument";
    case OCTGS_ENOSPC: return "workspace too small";
    case OCTGS_EHIP: return "HIP launch or runtime error";
    case OCTGS_EUNSUPPORTED: return "unsupported shape";
    default: return "unknown status";
  }
}

int octgs_version(void) { return 1; }

}  // extern "C"
