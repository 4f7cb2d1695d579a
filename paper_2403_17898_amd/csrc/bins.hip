// From grouped survivors to per-tile lists (the binning half of the forward
// rasterizer; Octree-GS Sec. III-A, tile-based front-to-back depth order).
//
// The projection leaves, per block of kSlots slots, the block's survivors
// grouped by screen bin.  Here:
//   k_bin_sort    one block per bin collects the bin's entries, sorts them by
//                 (depth bits, slot) in LDS, works out which of the bin's
//                 tiles each is listed in and counts the tiles' entries; a bin
//                 with more entries than one block sorts at once is put on a
//                 list instead;
//   k_tile_scan   first, by all its blocks together, those long bins: their
//                 entries to memory, then, a slice of the depths per block,
//                 sorted and counted; then the exclusive scan of the counts in
//                 tile order: each tile's range (and, in training, the blocks'
//                 pair numbers);
//   k_tile_lists  one block per bin writes its tiles' lists in depth order:
//                 a wave takes a tile and compacts the bin's ordered entries
//                 by ballots, so all writes are in place and in order; a long
//                 bin is done slice by slice.
// No sort pass over pairs, no look-back chain over hundreds of partitions: the
// waits on other blocks are the tile scan's (one block per 8,192 tiles) and,
// where there are long bins, those for units of work that running blocks have
// taken.  All are bounded.
#include "octgs_internal.h"

namespace octgs {

namespace {

constexpr int kNT = kBinThreads, kNW = kNT / kWave;
constexpr int kDigit = 9, kDigits = 1 << kDigit;  // radix of the block sort: one digit per thread
constexpr int kSeg = 4, kRound = kSeg * kNT;      // slot blocks per thread and round of collect
static_assert(kDigits == kNT, "one digit per thread");

constexpr int kTestBatch = kNT;  // long rectangles staged for their tile tests, one per thread

struct BinSmem {
  // entry p as collected: slot and tiles; its key is in kk[p] until the sort
  uint32_t su[kBinCap], mm[kBinCap];
  uint32_t kk[kBinCap];  // keys being sorted
  // positions being sorted, wave digit counters of a sort pass; before, where
  // the slot blocks' entries (and large survivors) start in the round, and
  // where in the blocks' groups
  union {
    struct {
      uint32_t vv[kBinCap];
      union {
        uint16_t wcnt[kNW][kDigits];
        struct {  // rectangles to test: 2D mean, conic, extent in the bin (4 bits each side)
          float mx[kTestBatch], my[kTestBatch], qa[kTestBatch], qb[kTestBatch], qc[kTestBatch];
          uint32_t box[kTestBatch];
        };
      };
    };
    struct {
      uint32_t pre[kRound], lpre[kRound];
      uint16_t first[kRound];
    };
  };
  uint32_t tmp[kNW], ltmp[kNW];
  uint32_t tcnt[32];
  unsigned long long cand;
  uint32_t vis, m, run, diff, flag, base, unknown, unit;
};

constexpr int kLarge = 4;  // large survivors looked at per thread at a time

// Index of the last of pre[0..kRound) that is <= i (pre[0] = 0, nondecreasing).
__device__ __forceinline__ uint32_t owner_of(const uint32_t *pre, uint32_t i) {
  uint32_t lo = 0;
#pragma unroll
  for (int st = kRound / 2; st > 0; st >>= 1)
    if (pre[lo + st] <= i) lo += st;
  return lo;
}

// All entries of a bin from slot blocks [b0, b1), in no particular order, handed
// to put(position, depth key, slot, tiles).  local: the bin's index in its band.
// Positions come from take(n): the first of n, asked for by one thread.  COUNT:
// positions count from 0 in sm.m, which ends as the number of entries; once they
// are more than kBinCap only that number is of use, and the grouped ones are not
// read; also the view's candidate and survivor counts into sm.cand and sm.vis.
// Everything that one slot block says about the bin is loaded at once, then all
// entries and large survivors: two dependent round trips for up to 2,048 blocks.
template <bool COUNT, typename Take, typename Put>
__device__ __forceinline__ void collect(const RasterWs &ws, BinSmem &sm, int local, uint32_t bx,
                                        uint32_t by, uint32_t b0, uint32_t b1, bool mine, Take take,
                                        Put put) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  if (COUNT && t == 0) {
    sm.m = 0u;
    sm.cand = 0ull;
    sm.vis = 0u;
  }
  uint64_t cand = 0;
  uint32_t vis = 0;
  for (uint32_t r0 = b0; r0 < b1; r0 += kRound) {
    uint32_t first[kSeg], c[kSeg], lc[kSeg], sc = 0, sl = 0;
#pragma unroll
    for (int j = 0; j < kSeg; ++j) {
      const uint32_t b = r0 + (uint32_t)(kSeg * t + j);
      const bool on = b < b1;
      const uint32_t bc = on ? b : b1 - 1u;  // unconditional loads, all in flight together
      const uint16_t *row = ws.group_off + (size_t)bc * ws.group_pitch + local;
      const uint32_t e0 = row[0], e1 = row[1], lg = ws.blk_large[bc];
      if (COUNT) {
        const uint32_t cv = ws.blk_cand[bc], vv = ws.blk_vis[bc];
        cand += on ? cv : 0u;
        vis += on ? vv : 0u;
      }
      first[j] = e0;
      c[j] = on && mine ? e1 - e0 : 0u;
      lc[j] = on && mine ? lg : 0u;
      sc += c[j];
      sl += lc[j];
    }
    // both exclusive scans at once
    const uint32_t is = wave_incl_scan(sc), il = wave_incl_scan(sl);
    if (l == kWave - 1) {
      sm.tmp[w] = is;
      sm.ltmp[w] = il;
    }
    __syncthreads();  // also: the last round's readers of pre, lpre and first are done
    uint32_t es = is - sc, el = il - sl, ts = 0, tl = 0;
#pragma unroll
    for (int v = 0; v < kNW; ++v) {
      if (v < w) {
        es += sm.tmp[v];
        el += sm.ltmp[v];
      }
      ts += sm.tmp[v];
      tl += sm.ltmp[v];
    }
    if (t == 0) sm.run = take(ts);
#pragma unroll
    for (int j = 0; j < kSeg; ++j) {
      sm.pre[kSeg * t + j] = es;
      sm.lpre[kSeg * t + j] = el;
      sm.first[kSeg * t + j] = (uint16_t)first[j];
      es += c[j];
      el += lc[j];
    }
    __syncthreads();
    const uint32_t run = sm.run;
    if (!(COUNT && run + ts > (uint32_t)kBinCap))
      for (uint32_t i = t; i < ts; i += kNT) {
        const uint32_t o = owner_of(sm.pre, i);
        const GroupEntry v = *group_entry(ws, r0 + o, sm.first[o] + (i - sm.pre[o]));
        put(run + i, v.key, v.slot, v.tiles);
      }
    // kLarge large survivors per thread at a time, their loads in flight together
    for (uint32_t i0 = w * kWave; i0 < tl; i0 += kLarge * kNT) {
      uint4 e[kLarge];
      uint64_t hm[kLarge];
      uint32_t n = 0;
#pragma unroll
      for (int u = 0; u < kLarge; ++u) {
        const uint32_t i = min(i0 + (uint32_t)(u * kNT + l), tl - 1u), o = owner_of(sm.lpre, i);
        e[u] = *group_large(ws, r0 + o, i - sm.lpre[o]);
      }
#pragma unroll
      for (int u = 0; u < kLarge; ++u) {
        const TileRect q = clip_to_bin(unpack_rect(e[u].x | ((uint64_t)e[u].y << 32)), ws.bins, bx, by);
        hm[u] = ballot(i0 + (uint32_t)(u * kNT + l) < tl && q.x0 < q.x1 && q.y0 < q.y1);
        n += (uint32_t)__popcll(hm[u]);
      }
      if (n == 0u) continue;
      uint32_t p = 0;
      if (l == 0) p = take(n);
      p = (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
#pragma unroll
      for (int u = 0; u < kLarge; ++u) {
        if ((hm[u] >> l) & 1ull)
          put(p + (uint32_t)__popcll(hm[u] & lanemask_lt()), e[u].z, e[u].w, kTilesUnknown);
        p += (uint32_t)__popcll(hm[u]);
      }
    }
    __syncthreads();
  }
  if (COUNT) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cand += __shfl_xor(cand, o, kWave);
    vis = wave_sum(vis);
    if (l == 0 && cand) atomicAdd(&sm.cand, (unsigned long long)cand);
    if (l == 0 && vis) atomicAdd(&sm.vis, vis);
    __syncthreads();
  }
}

// Puts the positions of the m collected entries into (key, slot) order in
// sm.vv (their keys, sorted, in sm.kk): a stable LSD radix sort by key, the
// entries in registers, striped (item j of wave w is entry 64 (w I + j) +
// lane), only over digits in which keys differ (depths of one bin share their
// exponent's high bits: three passes).  Ranking is a match-any by ballots per
// item; each wave owns a contiguous run, so equal digits keep their order.
// Entries arrive in no order, so equal keys (a few per bin: depths are floats)
// are put into slot order afterwards: short runs by the thread that owns the
// run's head; where a run is longer than kRun all entries are sorted by slot
// and then by the head of their run.
constexpr uint32_t kRun = 16;
constexpr int kPosBits = 12;
static_assert(kBinCap <= 1 << kPosBits, "positions and run heads share a word");

template <int I>
__device__ __forceinline__ void sort_entries(BinSmem &sm, uint32_t m) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const uint64_t lt = lanemask_lt();
  const uint32_t e0 = (uint32_t)(w * I * kWave + l);
  // phase 0: positions by key; phases 1 and 2, if needed: (run head, position)
  // by slot, then by run head
  for (int phase = 0; phase < 3; ++phase) {
    uint32_t key[I], val[I], d = 0;
#pragma unroll
    for (int j = 0; j < I; ++j) {
      const uint32_t e = min(e0 + (uint32_t)(j * kWave), m - 1u);
      if (phase == 0) {
        key[j] = sm.kk[e];
        val[j] = e;
      } else if (phase == 1) {
        const uint32_t p = sm.vv[e], k = sm.kk[e];
        uint32_t lo = 0, hi = e;  // first entry with this key
        while (lo < hi) {
          const uint32_t mid = (lo + hi) / 2;
          if (sm.kk[mid] < k) lo = mid + 1;
          else hi = mid;
        }
        key[j] = sm.su[p];
        val[j] = (lo << kPosBits) | p;
      } else {
        val[j] = sm.vv[e];
        key[j] = val[j] >> kPosBits;
      }
    }
    const uint32_t k0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)key[0]);
    if (t == 0) {
      sm.diff = 0u;
      sm.flag = 0u;
      sm.tmp[0] = k0;
    }
    lds_barrier();
    const uint32_t kf = sm.tmp[0];
#pragma unroll
    for (int j = 0; j < I; ++j) d |= key[j] ^ kf;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) d |= (uint32_t)__shfl_xor((int)d, o, kWave);
    if (l == 0 && d) atomicOr(&sm.diff, d);
    for (int i = t; i < kNW * kDigits / 2; i += kNT) reinterpret_cast<uint32_t *>(sm.wcnt)[i] = 0u;
    lds_barrier();
    const uint32_t diff = sm.diff;
    bool placed = false;
    for (int shift = 0; shift < 32; shift += kDigit) {
      if (((diff >> shift) & (kDigits - 1)) == 0u) continue;
      uint32_t rank[I];
#pragma unroll
      for (int j = 0; j < I; ++j) {
        const bool ok = e0 + (uint32_t)(j * kWave) < m;
        const uint32_t dg = (key[j] >> shift) & (kDigits - 1);
        uint64_t peers = ballot(ok);
#pragma unroll
        for (int b = 0; b < kDigit; ++b) {
          const int bit = (dg >> b) & 1;
          const uint64_t bal = ballot(bit);
          peers &= bit ? bal : ~bal;
        }
        uint32_t before = 0;
        if (ok) before = sm.wcnt[w][dg];
        // all lanes of the wave have read before any leader writes
        __builtin_amdgcn_wave_barrier();
        rank[j] = before + (uint32_t)__popcll(peers & lt);
        if (ok && (peers & lt) == 0ull)
          sm.wcnt[w][dg] = (uint16_t)(before + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
      }
      lds_barrier();
      // thread d owns digit d: its counts over the waves, then its start
      uint32_t cw[kNW], tot = 0, all;
#pragma unroll
      for (int v = 0; v < kNW; ++v) cw[v] = sm.wcnt[v][t];
#pragma unroll
      for (int v = 0; v < kNW; ++v) {
        const uint32_t c = cw[v];
        cw[v] = tot;
        tot += c;
      }
      const uint32_t st = block_scan<kNT>(tot, sm.tmp, &all);
#pragma unroll
      for (int v = 0; v < kNW; ++v) sm.wcnt[v][t] = (uint16_t)(cw[v] + st);
      lds_barrier();
#pragma unroll
      for (int j = 0; j < I; ++j) {
        if (e0 + (uint32_t)(j * kWave) < m) {
          const uint32_t pos = sm.wcnt[w][(key[j] >> shift) & (kDigits - 1)] + rank[j];
          sm.kk[pos] = key[j];
          sm.vv[pos] = val[j];
        }
      }
      lds_barrier();
#pragma unroll
      for (int j = 0; j < I; ++j) {
        const uint32_t e = min(e0 + (uint32_t)(j * kWave), m - 1u);
        key[j] = sm.kk[e];
        val[j] = sm.vv[e];
      }
#pragma unroll
      for (int v = 0; v < kNW; ++v) sm.wcnt[v][t] = 0;
      lds_barrier();
      placed = true;
    }
    if (!placed) {  // all keys equal: the entries keep their order
#pragma unroll
      for (int j = 0; j < I; ++j) {
        const uint32_t e = e0 + (uint32_t)(j * kWave);
        if (e < m) {
          sm.kk[e] = key[j];
          sm.vv[e] = val[j];
        }
      }
      lds_barrier();
    }
    if (phase == 0) {
      for (uint32_t i = t; i + 1 < m; i += kNT) {
        const uint32_t k = sm.kk[i];
        if (sm.kk[i + 1] != k || (i > 0 && sm.kk[i - 1] == k)) continue;
        uint32_t e = i + 2;
        while (e < m && e - i <= kRun && sm.kk[e] == k) ++e;
        if (e - i > kRun) {
          sm.flag = 1u;
          continue;
        }
        for (uint32_t a = i + 1; a < e; ++a) {  // insertion sort
          const uint32_t v = sm.vv[a], sv = sm.su[v];
          uint32_t b = a;
          for (; b > i && sm.su[sm.vv[b - 1]] > sv; --b) sm.vv[b] = sm.vv[b - 1];
          sm.vv[b] = v;
        }
      }
      lds_barrier();
      if (!sm.flag) break;
      lds_barrier();  // everyone has read the flag before it is cleared
    }
  }
}

__device__ __forceinline__ void sort_any(BinSmem &sm, uint32_t m) {
  static_assert(kBinItems == 8, "item counts of the sort");
  if (m <= kNT) sort_entries<1>(sm, m);
  else if (m <= 2 * kNT) sort_entries<2>(sm, m);
  else if (m <= 4 * kNT) sort_entries<4>(sm, m);
  else sort_entries<8>(sm, m);
}

// The tiles of the collected entries [0, cm) that came without them, and the
// number of entries per tile of the bin (lane j: tile j) of the wave's share.
// The unknown ones (long rectangles, up to a third of a bin and next to each
// other) are listed first (in sm.vv, unused until the sort); then a wave takes
// as many entries as it has lanes for, a tile per lane, so that all lanes and
// waves share them.  (With half a wave per entry, and one large survivor per
// thread at a time in collect, 15,000 Gaussians of 30 to 180 px in 512 x 512, most
// of them over more than 16 bins of 2 x 2 tiles, took 141 us here; now 57.)
__device__ __forceinline__ uint32_t finish_tiles(const RasterWs &ws, BinSmem &sm, uint32_t cm,
                                                 uint32_t bx, uint32_t by) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const BinGrid &bg = ws.bins;
  if (t == 0) sm.unknown = 0u;
  lds_barrier();
  for (uint32_t i0 = w * kWave; i0 < cm; i0 += kNT) {
    const uint32_t i = i0 + l;
    const bool un = i < cm && sm.mm[i] == kTilesUnknown;
    const uint64_t um = ballot(un);
    if (um == 0ull) continue;
    uint32_t p = 0;
    if (l == 0) p = atomicAdd(&sm.unknown, (uint32_t)__popcll(um));
    p = (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
    if (un) sm.vv[p + (uint32_t)__popcll(um & lanemask_lt())] = i;
  }
  lds_barrier();
  const uint32_t nu = sm.unknown;
  // a lane per tile of the bin, 64 / (tiles of the bin) entries per wave
  const int lgt = bg.sx + bg.sy, tl = l & ((1 << lgt) - 1);
  const uint32_t tx = (uint32_t)(tl & ((1 << bg.sx) - 1)), ty = (uint32_t)(tl >> bg.sx);
  const uint32_t step = (uint32_t)kWave >> lgt, tiles = (uint32_t)((1ull << (1 << lgt)) - 1ull);
  for (uint32_t k0 = 0; k0 < nu; k0 += kTestBatch) {
    const uint32_t nk = min(nu - k0, (uint32_t)kTestBatch);
    if ((uint32_t)t < nk) {
      const uint32_t i = sm.vv[k0 + t], slot = sm.su[i];
      const ulonglong2 rm = ws.rect[slot];
      const float4 A = ws.proj[3 * (size_t)slot], Q = ws.proj[3 * (size_t)slot + 2];
      const TileRect r = unpack_rect(rm.x), c = clip_to_bin(r, bg, bx, by);
      uint32_t box = (c.x0 - (bx << bg.sx)) | ((c.x1 - (bx << bg.sx)) << 4) |
                     ((c.y0 - (by << bg.sy)) << 8) | ((c.y1 - (by << bg.sy)) << 12);
      if (rect_tiles(r) <= kKeepBits) {  // known after all: nothing to test
        sm.mm[i] = bin_tiles(r, rm.y, bg, bx, by);
        box = ~0u;
      }
      sm.mx[t] = A.x;
      sm.my[t] = A.y;
      sm.qa[t] = Q.y;
      sm.qb[t] = Q.z;
      sm.qc[t] = Q.w;
      sm.box[t] = box;
    }
    lds_barrier();
    for (uint32_t j = step * w; j < nk; j += step * kNW) {
      const uint32_t e = min(j + (uint32_t)(l >> lgt), nk - 1u);
      const uint32_t box = sm.box[e];
      const bool in = tx >= (box & 15u) && tx < ((box >> 4) & 15u) && ty >= ((box >> 8) & 15u) &&
                      ty < ((box >> 12) & 15u);
      const bool hit = in && tile_meets_ellipse(sm.mx[e], sm.my[e], sm.qa[e], sm.qb[e], sm.qc[e],
                                                (bx << bg.sx) + tx, (by << bg.sy) + ty, ws.xmax,
                                                ws.ymax);
      const uint64_t hm = ballot(hit);
      if (tl == 0 && box != ~0u) sm.mm[sm.vv[k0 + e]] = (uint32_t)(hm >> l) & tiles;
    }
    lds_barrier();
  }
  // per wave and tile a scalar count (bits of tiles that the bin does not have
  // are clear)
  uint32_t cnt[32];
#pragma unroll
  for (int j = 0; j < 32; ++j) cnt[j] = 0u;
  lds_barrier();
  for (uint32_t i0 = w * kWave; i0 < cm; i0 += kNT) {
    const uint32_t i = i0 + l;
    const uint32_t bits = i < cm ? sm.mm[i] : 0u;
#pragma unroll
    for (int j = 0; j < 32; ++j) cnt[j] += (uint32_t)__popcll(ballot((bits & (1u << j)) != 0u));
  }
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < 32; ++j) mine = l == j ? cnt[j] : mine;
  return mine;
}

// One block per bin of the band.  Bound by latency: the collection's two
// memory round trips, the test of long rectangles, about 20 LDS barriers of
// the sort (lists of a few hundred to a thousand entries, three digit passes):
// on a 1920 x 1080 view of 862k pairs a block takes 18 us (collection 5.7,
// listing and testing long rectangles 6.3, counts 1.3, sort 4, writes 1.4) and
// the kernel 21; on 3840 x 2160 there are two rounds of blocks, 49.  (With the
// long bins' runs in this kernel its registers spilled: 25 and 60.)
__global__ __launch_bounds__(kNT, 4) void k_bin_sort(RasterWs ws, int band_row0, uint32_t nband) {
  __shared__ BinSmem sm;
  const uint32_t item = xcd_item(blockIdx.x, nband);
  if (item >= nband) return;
  const int t = threadIdx.x, l = __lane_id();
  const BinGrid &bg = ws.bins;
  const uint32_t bx = item % (uint32_t)bg.nx;
  const uint32_t by = (uint32_t)band_row0 + item / (uint32_t)bg.nx;
  const uint32_t bin = by * (uint32_t)bg.nx + bx;
  const uint32_t nblk = slot_blocks(ws.hdr->n_slots);
  const bool reach = bx < (uint32_t)bg.gx;
  const int local = reach ? (int)((by - (uint32_t)band_row0) * (uint32_t)bg.gx + bx) : 0;
  if (t < 32) sm.tcnt[t] = 0u;
  collect<true>(
      ws, sm, local, bx, by, 0u, nblk, reach, [&](uint32_t n) { return atomicAdd(&sm.m, n); },
      [&](uint32_t p, uint32_t key, uint32_t slot, uint32_t tiles) {
        if (p < (uint32_t)kBinCap) {
          sm.kk[p] = key;
          sm.su[p] = slot;
          sm.mm[p] = tiles;
        }
      });
  // candidates of the whole view: nothing is listed if they exceed the capacity
  const uint32_t cand = (uint32_t)std::min<uint64_t>(sm.cand, kLbVal);
  const bool over = cand > (uint64_t)ws.pcap;
  if (bin == 0 && t == 0) {
    ws.hdr->n_visible = sm.vis;
    ws.hdr->n_candidates = cand;
    ws.hdr->pair_overflow = over ? 1u : 0u;
  }
  const uint32_t m = over ? 0u : sm.m;
  // (every entry stands for at least one candidate tile of its own, so the lists
  // of all bins fit the capacity)
  if (m > (uint32_t)kBinCap) {
    // a long bin: its place and its slices; its entries to memory, or, if they
    // are many, on the list of those that all blocks copy
    const uint32_t ns = long_slices(m);
    if (t == 0) {
      sm.base = atomicAdd(&ws.hdr->bin_cursor, m);
      sm.unit = atomicAdd(&ws.hdr->n_slices, ns);
      ws.bin_range[bin] = make_uint2(sm.base, m);
      if (m > kCopyCap) {
        const uint32_t q = atomicAdd(&ws.hdr->n_over, 1u);
        ws.over_bin[2 * q] = bin;
        ws.over_bin[2 * q + 1] = 0u;
      }
    }
    __syncthreads();
    if (t == 0) sm.m = 0u;
    for (uint32_t i = t; i < ns; i += kNT) {
      ws.slices[kSliceRow * (size_t)(sm.unit + i)] = bin;
      ws.slices[kSliceRow * (size_t)(sm.unit + i) + 1] = i;
    }
    if (m <= kCopyCap) {
      const uint32_t gb = sm.base;
      collect<false>(
          ws, sm, local, bx, by, 0u, nblk, reach, [&](uint32_t n) { return atomicAdd(&sm.m, n); },
          [&](uint32_t p, uint32_t key, uint32_t slot, uint32_t tiles) {
            ws.tkey[gb + p] = key;
            ws.bin_slot[0][gb + p] = slot;
            ws.bin_mask[0][gb + p] = tiles;
          });
    }
  } else if (m > 0) {
    const uint32_t mine = finish_tiles(ws, sm, m, bx, by);
    // all bins ask at about the same time, and the answers come one after
    // the other: the sort, which loads nothing, covers the wait
    uint32_t base = 0;
    if (t == 0) base = atomicAdd(&ws.hdr->bin_cursor, m);
    sort_any(sm, m);
    if (t == 0) {
      sm.base = base;
      ws.bin_range[bin] = make_uint2(base, m);
    }
    if (l < 32 && mine) atomicAdd(&sm.tcnt[l], mine);
    lds_barrier();
    const uint32_t gb = sm.base;
    for (uint32_t i = t; i < m; i += kNT) {
      const uint32_t p = sm.vv[i] & ((1u << kPosBits) - 1u);
      ws.bin_slot[0][gb + i] = sm.su[p];
      ws.bin_mask[0][gb + i] = sm.mm[p];
    }
  } else if (t == 0) {
    ws.bin_range[bin] = make_uint2(0u, 0u);
  }
  lds_barrier();
  if (t < (1 << (bg.sx + bg.sy))) {
    const uint32_t tx = (bx << bg.sx) + (t & ((1u << bg.sx) - 1u)), ty = (by << bg.sy) + (t >> bg.sx);
    if (tx < (uint32_t)ws.tiles_x && ty < (uint32_t)ws.tiles_y)
      ws.tile_count[(size_t)ty * ws.tiles_x + tx] = sm.tcnt[t];
  }
}

// ---- long bins --------------------------------------------------------------
// Bins of more than kBinCap entries, done by all blocks of the scan kernel
// together in two phases of units, each taken by the next free block: first
// the entries of those that are too many for the bin's block to copy (a unit:
// one bin's from some slot blocks), then the slices of their depths.  A block
// that finds no more units waits for those that are taken, which running blocks
// work on: no wait is on a block that has not started.
// Bound by latency: about 20 us for the copies and 35 for a block's slice (sample
// 7, pass over the bin's keys 5 for 5,000 of them, tile tests 5, sort 9), more of
// it for the pass where a bin has 100k entries.  300k Gaussians, projection and
// binning (us), with two global sorts / one block per bin and a merge by rank /
// now: within 64 x 64 px 176 / 4,700 / 246, 200 x 200 175 / - / 203, 400 x 400
// 175 / 290 / 171, 600 x 600 174 / - / 130.  Four 1080p views in flight, 64 bins
// of 4 to 8 thousand entries among 1,020: 961 with the merge, 945 now (1,020
// where all long bins were copied in the first phase).  256 blocks for them: with
// 64 and 128, 500 and 360 instead of 270 within 64 x 64 px.  Four waves per SIMD
// although that spills: at 207 registers the blocks, there in every view, made
// four 1080p views in flight 2 to 4 percent slower.

// Waits (thread 0) until *done reaches want; false if the wait hit its bound
// (then *err is set).  What was written before the counts is visible after it.
__device__ __forceinline__ bool wait_units(BinSmem &sm, const uint32_t *done, uint32_t want,
                                           uint32_t *err) {
  if (threadIdx.x == 0) {
    uint32_t spins = 0;
    while (ld_acq(done) < want && ++spins <= kSpinLimit) __builtin_amdgcn_s_sleep(1);
    sm.flag = spins <= kSpinLimit ? 1u : 0u;
    if (!sm.flag) atomicOr(err, 1u);
  }
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // every wave, for its own loads
  const bool ok = sm.flag != 0u;
  __syncthreads();
  return ok;
}

// Units [0, total) by work(unit), as many as this block gets, then their number
// is added to *done.  A barrier does not wait for the waves' stores and atomics,
// so each wave waits for its own before the barrier that leads to the count.
// STORES: other blocks read what the units store, so the XCD's L2, where the
// stores are by then, is written back; atomics are done in memory (all eight
// waves writing it back took 10 to 30 us more).
constexpr int kVmcnt0 = 0x0f70;  // s_waitcnt operand: vmcnt(0), the other counters as they are
template <bool STORES, typename Work>
__device__ __forceinline__ void take_units(BinSmem &sm, uint32_t *next, uint32_t *done,
                                           uint32_t total, Work work) {
  uint32_t n = 0;
  for (;; ++n) {
    if (threadIdx.x == 0) sm.unit = atomicAdd(next, 1u);
    __syncthreads();
    const uint32_t u = sm.unit;
    if (u >= total) break;
    work(u);
    __syncthreads();  // the LDS may be reused
  }
  if (n == 0) return;
  __builtin_amdgcn_s_waitcnt(kVmcnt0);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (STORES) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      // the fence's own wait is dropped where nothing but its write-back is counted
      __builtin_amdgcn_s_waitcnt(kVmcnt0);
    }
    atomicAdd(done, n);
  }
}

// One unit of the first phase: entries of long bin q (of the band from bin row
// band_row0 on) from slot blocks [b0, b1).
__device__ __forceinline__ void long_copy(const RasterWs &ws, BinSmem &sm, uint32_t q, uint32_t b0,
                                          uint32_t b1, uint32_t band_row0) {
  const BinGrid &bg = ws.bins;
  const uint32_t bin = ws.over_bin[2 * q], bx = bin % (uint32_t)bg.nx, by = bin / (uint32_t)bg.nx;
  const uint32_t gb = ws.bin_range[bin].x;
  collect<false>(
      ws, sm, (int)((by - band_row0) * (uint32_t)bg.gx + bx), bx, by, b0, b1,
      true, [&](uint32_t n) { return atomicAdd(&ws.over_bin[2 * q + 1], n); },
      [&](uint32_t p, uint32_t key, uint32_t slot, uint32_t tiles) {
        ws.tkey[gb + p] = key;
        ws.bin_slot[0][gb + p] = slot;
        ws.bin_mask[0][gb + p] = tiles;
      });
}

// Entries of a long bin whose (key, slot) lie in [lo, hi): their positions into
// sm.su while there are no more than kBinCap, their number, and in sm.vis the
// number of those before lo.  Reads all keys (slots only where a key equals a
// bound's), eight loads per thread in flight, a step ahead of their use.
__device__ __forceinline__ uint32_t pick(BinSmem &sm, const uint32_t *key, const uint32_t *slot,
                                         uint32_t m, uint64_t lo, uint64_t hi) {
  constexpr int kU = 8;
  const int t = threadIdx.x, l = __lane_id();
  const uint32_t klo = (uint32_t)(lo >> 32), khi = (uint32_t)(hi >> 32);
  __syncthreads();  // the last readers of sm.m and sm.vis
  if (t == 0) sm.m = sm.vis = 0u;
  __syncthreads();
  uint32_t before = 0, next[kU];
  auto load = [&](uint32_t e0) {
#pragma unroll
    for (int u = 0; u < kU; ++u) next[u] = key[min(e0 + (uint32_t)(u * kNT + t), m - 1u)];
  };
  load(0u);
  for (uint32_t e0 = 0; e0 < m; e0 += kU * kNT) {
    uint64_t v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t e = e0 + (uint32_t)(u * kNT + t);
      v[u] = (uint64_t)next[u] << 32;
      if (next[u] == klo || next[u] == khi) v[u] |= slot[min(e, m - 1u)];
    }
    load(min(e0 + (uint32_t)(kU * kNT), m - 1u));
    uint64_t im[kU];
    uint32_t n = 0;
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const bool on = e0 + (uint32_t)(u * kNT + t) < m;
      before += on && v[u] < lo ? 1u : 0u;
      im[u] = ballot(on && v[u] >= lo && v[u] < hi);
      n += (uint32_t)__popcll(im[u]);
    }
    if (n == 0u) continue;
    uint32_t p = 0;
    if (l == 0) p = atomicAdd(&sm.m, n);
    p = (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const uint32_t at = p + (uint32_t)__popcll(im[u] & lanemask_lt());
      if (((im[u] >> l) & 1ull) && at < (uint32_t)kBinCap) sm.su[at] = e0 + (uint32_t)(u * kNT + t);
      p += (uint32_t)__popcll(im[u]);
    }
  }
  before = wave_sum(before);
  if (l == 0 && before) atomicAdd(&sm.vis, before);
  __syncthreads();
  return sm.m;
}

// One unit of the second phase: slice `unit` of a long bin, the entries between
// two of the splitters that divide an even sample of the bin into its slices.
// (key, slot) differs for all entries, so the slices are a partition whatever
// the keys, every block that works on one bin sorts the same sample, and none
// needs another's result: the entries before the slice are counted.  A slice
// that is more than a block sorts at once (the sample's luck, or more slices
// than samples) is halved until it is not.
__device__ __forceinline__ void long_slice(const RasterWs &ws, BinSmem &sm, uint32_t unit) {
  const int t = threadIdx.x, l = __lane_id();
  const BinGrid &bg = ws.bins;
  uint32_t *row = ws.slices + kSliceRow * (size_t)unit;
  const uint32_t bin = row[0], s = row[1];
  const uint32_t bx = bin % (uint32_t)bg.nx, by = bin / (uint32_t)bg.nx;
  const uint2 rg = ws.bin_range[bin];
  const uint32_t m = rg.y, ns = long_slices(m);
  const uint32_t *key = ws.tkey + rg.x, *slot = ws.bin_slot[0] + rg.x, *mask = ws.bin_mask[0] + rg.x;
  // 64 samples a slice, but no more than 2,048 in all (m > kBinCap, so they differ)
  const int lg = ns <= 8u ? 9 : (ns <= 16u ? 10 : 11);
  uint32_t c = 1u << lg;
  for (uint32_t i = t; i < c; i += kNT) {
    const uint32_t e = (uint32_t)(((uint64_t)i * m) >> lg);
    sm.kk[i] = key[e];
    sm.su[i] = slot[e];
  }
  if (t < 32) sm.tcnt[t] = 0u;
  auto splitter = [&](uint32_t i) -> uint64_t {
    const uint32_t p = (uint32_t)(((uint64_t)i << lg) / ns);
    return ((uint64_t)sm.kk[p] << 32) | sm.su[sm.vv[p] & ((1u << kPosBits) - 1u)];
  };
  uint64_t lo = 0, hi = 0;
  uint32_t pos = 0, size = 0, mine = 0, at = 0;
  // the sample, then the slice (in as many parts as it takes)
  for (bool sample = true;; sample = false) {
    lds_barrier();
    if (!sample && c) mine += finish_tiles(ws, sm, c, bx, by);
    if (c) sort_any(sm, c);
    lds_barrier();
    if (sample) {
      lo = s > 0u ? splitter(s) : 0ull;
      hi = s + 1u < ns ? splitter(s + 1u) : ~0ull;
    } else {
      for (uint32_t i = t; i < c; i += kNT) {
        const uint32_t p = sm.vv[i] & ((1u << kPosBits) - 1u);
        ws.bin_slot[1][rg.x + at + i] = sm.su[p];
        ws.bin_mask[1][rg.x + at + i] = sm.mm[p];
      }
      if (lo >= hi) break;
    }
    uint64_t h = hi;
    c = pick(sm, key, slot, m, lo, h);
    while (c > (uint32_t)kBinCap) {
      h = lo + (h - lo) / 2u;
      c = pick(sm, key, slot, m, lo, h);
    }
    at = sm.vis;
    if (sample) pos = at;
    lo = h;
    size += c;
    for (uint32_t i = t; i < c; i += kNT) {
      const uint32_t e = sm.su[i];
      sm.kk[i] = key[e];
      sm.su[i] = slot[e];
      sm.mm[i] = mask[e];
    }
  }
  if (l < 32 && mine) atomicAdd(&sm.tcnt[l], mine);
  __syncthreads();
  if (t == 0) {
    row[2] = pos;
    row[3] = size;
  }
  if (t < 32) {
    row[4 + t] = sm.tcnt[t];
    const uint32_t tx = (bx << bg.sx) + (t & ((1u << bg.sx) - 1u)), ty = (by << bg.sy) + (t >> bg.sx);
    if (sm.tcnt[t]) atomicAdd(&ws.tile_count[(size_t)ty * ws.tiles_x + tx], sm.tcnt[t]);
  }
}

// The first phase alone, where bands of bin rows share the groups.
__global__ __launch_bounds__(kNT) void k_long_copy(RasterWs ws, int band_row0, int rows) {
  __shared__ BinSmem sm;
  const uint32_t nblk = slot_blocks(ws.hdr->n_slots), nover = ws.hdr->n_over;
  for (uint32_t q = 0; q < nover; ++q) {
    const uint32_t by = ws.over_bin[2 * q] / (uint32_t)ws.bins.nx;
    if (by < (uint32_t)band_row0 || by >= (uint32_t)(band_row0 + rows)) continue;
    for (uint32_t b0 = blockIdx.x * kLongSeg; b0 < nblk; b0 += gridDim.x * kLongSeg) {
      __syncthreads();
      long_copy(ws, sm, q, b0, min(b0 + kLongSeg, nblk), (uint32_t)band_row0);
    }
  }
}

constexpr int kLongBlocks = 256;  // blocks that are there for long bins only

// Slot blocks per unit of the first phase: about a unit per block.
__device__ __forceinline__ uint32_t long_seg(uint32_t nover, uint32_t nblk) {
  const uint64_t all = (uint64_t)nover * nblk;
  return (uint32_t)min((all + kLongBlocks - 1u) / kLongBlocks + kLongSeg - 1u, (uint64_t)nblk);
}

// Long bins first (COPIED: their entries are in memory already).  Then:
// Blocks [0, scan): ranges of kScanThreads * kScanTiles consecutive tiles each, chained
// by decoupled look-back; the block number is a ticket taken in the order
// blocks start, so every block that one waits on is already running.
// Block scan: pair numbers of the slot blocks (training).
__global__ __launch_bounds__(kScanThreads, 4) void k_tile_scan(RasterWs ws, int train, int copied) {
  static_assert(kScanThreads == kNT, "long bins are done by the same blocks");
  __shared__ BinSmem sm;
  __shared__ uint32_t s_b, s_excl;
  uint32_t *tmp = sm.tmp;
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  bool ok = true;
  const uint32_t ns = ws.hdr->n_slices;
  if (ns > 0u) {
    const uint32_t nover = copied ? 0u : ws.hdr->n_over;
    if (nover > 0u) {
      const uint32_t nblk = slot_blocks(ws.hdr->n_slots), seg = long_seg(nover, nblk);
      const uint32_t per = (nblk + seg - 1u) / seg;
      take_units<true>(sm, &ws.hdr->copy_next, &ws.hdr->copy_done, nover * per, [&](uint32_t u) {
        const uint32_t b0 = u % per * seg;
        long_copy(ws, sm, u / per, b0, min(b0 + seg, nblk), 0u);
      });
      ok = wait_units(sm, &ws.hdr->copy_done, nover * per, &ws.hdr->sync_error);
    }
    if (ok)
      // (only their counts, added by atomics, are read in this kernel)
      take_units<false>(sm, &ws.hdr->slice_next, &ws.hdr->slice_done, ns,
                        [&](uint32_t u) { long_slice(ws, sm, u); });
    // (blocks that are there for the long bins need not wait)
    if (blockIdx.x < (uint32_t)ws.scan_blocks)
      ok = wait_units(sm, &ws.hdr->slice_done, ns, &ws.hdr->sync_error) && ok;
  }
  if (blockIdx.x < (uint32_t)ws.scan_blocks) {
    if (t == 0) s_b = ws.scan_blocks > 1 ? atomicAdd(&ws.hdr->scan_ticket, 1u) : 0u;
    __syncthreads();
    const uint32_t b = s_b;
    const int64_t ntiles = (int64_t)ws.tiles_x * ws.tiles_y;
    const int64_t t0 = ((int64_t)b * kScanThreads + t) * kScanTiles;
    uint32_t c[kScanTiles], sum = 0;
    // the count array is padded to whole blocks; words past the last tile are
    // not counts
    const uint4 *src = reinterpret_cast<const uint4 *>(ws.tile_count + t0);
#pragma unroll
    for (int q = 0; q < kScanTiles / 4; ++q) {
      const uint4 v = src[q];
      c[4 * q] = v.x; c[4 * q + 1] = v.y; c[4 * q + 2] = v.z; c[4 * q + 3] = v.w;
    }
#pragma unroll
    for (int q = 0; q < kScanTiles; ++q) {
      // (no lists at all if a wait hit its bound)
      if (t0 + q >= ntiles || !ok) c[q] = 0u;
      sum += c[q];
    }
    uint32_t tot;
    uint32_t run = block_scan<kScanThreads>(sum, tmp, &tot);
    if (w == 0) {
      const uint32_t ex = ws.scan_blocks > 1
                              ? chained_lookback(ws.lb_scan, b, tot, &ws.hdr->sync_error, kSpinLimit)
                              : 0u;
      if (l == 0) s_excl = ex;
    }
    __syncthreads();
    run += s_excl;
    uint2 *out = reinterpret_cast<uint2 *>(ws.ranges) + t0;
#pragma unroll
    for (int q = 0; q < kScanTiles; ++q) {
      if (t0 + q < ntiles) out[q] = c[q] ? make_uint2(run, run + c[q]) : make_uint2(0u, 0u);
      run += c[q];
    }
    if (b == (uint32_t)ws.scan_blocks - 1 && t == 0) {
      ws.hdr->n_listed = s_excl + tot;
      ws.hdr->n_pairs = s_excl + tot;
    }
    return;
  }
  if (blockIdx.x == (uint32_t)ws.scan_blocks && train) {
    const uint32_t nblk = slot_blocks(ws.hdr->n_slots);
    uint32_t run = 0;
    for (uint32_t r0 = 0; r0 < nblk; r0 += kScanThreads) {
      const uint32_t b = r0 + t;
      uint32_t tot;
      const uint32_t ex = block_scan<kScanThreads>(b < nblk ? ws.blk_pairs[b] : 0u, tmp, &tot);
      if (b < nblk) ws.blk_pairs[b] = run + ex;
      run += tot;
    }
    if (t == 0) ws.hdr->n_emit = ws.hdr->pair_overflow ? 0u : run;
  }
}

constexpr int kOrderBuckets = 64;  // = kWave: one scan lane per bucket

// Half-octave bucket of a tile's list length, longest lists first; empty
// tiles and blocks without a tile go last (kOrderBuckets - 1).
__device__ __forceinline__ uint32_t order_bucket(int32_t tile, const uint32_t *ranges) {
  if (tile < 0) return kOrderBuckets - 1;
  const uint32_t len = ranges[2 * tile + 1] - ranges[2 * tile];
  if (len == 0) return kOrderBuckets - 1;
  const uint32_t lg = 31u - (uint32_t)__clz(len);
  const uint32_t half = lg > 0 ? (len >> (lg - 1)) & 1u : 0u;
  return (uint32_t)(kOrderBuckets - 2) - min(2u * lg + half, (uint32_t)(kOrderBuckets - 2));
}

constexpr int kLT = 512, kLW = kLT / kWave;  // threads and waves of the list kernel
constexpr int kLStage = 2048;                // entries staged in LDS at a time

struct OrderSmem {
  uint32_t cnt[kOrderBuckets];
  uint32_t wcnt[kLW][kOrderBuckets];
  uint32_t run[kOrderBuckets];
};

// Block x of the order blocks takes the slots that the group mapping gives XCD
// x and writes their tiles to tile_order[x + 8 * position] in a stable order by
// bucket (longest lists first): a counting pass, then chunks of slots ranked
// per wave with ballots (match-any on the bucket bits), each wave owning a
// contiguous run.  Every position of the XCD is written once, so tile_order is
// a permutation of the group mapping.
__device__ __forceinline__ void order_tiles(const RasterWs &ws, uint32_t xcd, OrderSmem &sm) {
  constexpr int kItems = 4;
  const uint32_t nslots = tile_grid_blocks(ws.tiles_x, ws.tiles_y) / kXcds;
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const uint64_t lt = lanemask_lt();
  if (xcd == 0 && t == 0) ws.hdr->tile_ordered = 1u;
  if (t < kOrderBuckets) sm.cnt[t] = 0u;
  __syncthreads();
  for (uint32_t q = t; q < nslots; q += kLT)
    atomicAdd(&sm.cnt[order_bucket(tile_of_block(xcd + kXcds * q, ws.tiles_x, ws.tiles_y),
                                   ws.ranges)], 1u);
  __syncthreads();
  if (w == 0) {
    const uint32_t v = sm.cnt[l];
    sm.run[l] = wave_incl_scan(v) - v;
  }
  for (uint32_t c0 = 0; c0 < nslots; c0 += kLT * kItems) {
    (&sm.wcnt[0][0])[t] = 0u;  // kLW * kOrderBuckets == kLT
    int32_t tl[kItems];
    uint32_t key[kItems], rank[kItems];
    bool ok[kItems];
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      const uint32_t q = c0 + (uint32_t)(w * kWave * kItems + j * kWave + l);
      ok[j] = q < nslots;
      tl[j] = ok[j] ? tile_of_block(xcd + kXcds * q, ws.tiles_x, ws.tiles_y) : -1;
      key[j] = order_bucket(tl[j], ws.ranges);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j) {
      uint64_t peers = ballot(ok[j]);
#pragma unroll
      for (int b = 0; b < 6; ++b) {
        const int bit = (key[j] >> b) & 1;
        const uint64_t bal = ballot(bit);
        peers &= bit ? bal : ~bal;
      }
      uint32_t before = 0;
      if (ok[j]) before = sm.wcnt[w][key[j]];
      // all lanes of the wave have read before any leader writes
      __builtin_amdgcn_wave_barrier();
      if (ok[j]) {
        rank[j] = before + (uint32_t)__popcll(peers & lt);
        if ((peers & lt) == 0) sm.wcnt[w][key[j]] = before + (uint32_t)__popcll(peers);
      }
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    if (t < kOrderBuckets) {
      uint32_t base = sm.run[t];
#pragma unroll
      for (int v = 0; v < kLW; ++v) {
        const uint32_t c = sm.wcnt[v][t];
        sm.wcnt[v][t] = base;
        base += c;
      }
      sm.run[t] = base;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kItems; ++j)
      if (ok[j]) ws.tile_order[xcd + kXcds * (sm.wcnt[w][key[j]] + rank[j])] = (uint32_t)tl[j];
    __syncthreads();
  }
}

template <bool TRAIN>
struct ListSmem {
  uint32_t slot[kLStage], mask[kLStage];
  // training: staged entries whose rectangles number all their tiles
  uint32_t first[TRAIN ? kLStage : 1], org[TRAIN ? kLStage : 1], end[TRAIN ? kLStage : 1];
  uint16_t index[TRAIN ? kLStage : 1];
  uint32_t nfull;
};

constexpr int kTilesPerWave = 32 / kLW;

// The tiles of a bin that a wave writes the lists of, and where in them it is.
struct ListTiles {
  uint32_t tile[kTilesPerWave], run[kTilesPerWave];
  bool on[kTilesPerWave];
};

__device__ __forceinline__ ListTiles list_tiles(const RasterWs &ws, uint32_t bx, uint32_t by, int w) {
  const BinGrid &bg = ws.bins;
  const int nt = 1 << (bg.sx + bg.sy);
  ListTiles r;
#pragma unroll
  for (int q = 0; q < kTilesPerWave; ++q) {
    const int j = w + q * kLW;
    const uint32_t tx = (bx << bg.sx) + (uint32_t)(j & ((1 << bg.sx) - 1));
    const uint32_t ty = (by << bg.sy) + (uint32_t)(j >> bg.sx);
    r.on[q] = j < nt && tx < (uint32_t)ws.tiles_x && ty < (uint32_t)ws.tiles_y;
    r.tile[q] = ty * (uint32_t)ws.tiles_x + tx;
    r.run[q] = r.on[q] ? ws.ranges[2 * (size_t)r.tile[q]] : 0u;
  }
  return r;
}

// Appends n ordered entries of bin (bx, by) to its tiles' lists.  The entries are
// staged in LDS kLStage at a time; each wave walks them for up to four of the
// bin's tiles and appends those whose mask has the tile's bit.
// Training: rectangles with more than kKeepBits tiles number all their tiles
// as pairs; the rows of the numbers without a pair are cleared here, half a
// wave per entry, a tile per lane.
template <bool TRAIN>
__device__ __forceinline__ void append(const RasterWs &ws, ListSmem<TRAIN> &ls, ListTiles &lt,
                                       const uint32_t *slots, const uint32_t *masks, uint32_t n,
                                       uint32_t bx, uint32_t by, uint32_t nblk) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const uint64_t lmask = lanemask_lt();
  const BinGrid &bg = ws.bins;
  const int nt = 1 << (bg.sx + bg.sy);
  for (uint32_t c0 = 0; c0 < n; c0 += kLStage) {
    const uint32_t cm = min((uint32_t)kLStage, n - c0);
    __syncthreads();
    if (TRAIN) {
      if (t == 0) ls.nfull = 0u;
      __syncthreads();
    }
    for (uint32_t i = t; i < cm; i += kLT) {
      const uint32_t s = slots[c0 + i];
      ls.slot[i] = s;
      ls.mask[i] = masks[c0 + i];
      if (TRAIN) {
        const uint64_t rc = ws.rect[s].x;
        const uint32_t first = ws.blk_pairs[slot_block(s, nblk)] + ws.pair_base[s];
        if (rect_tiles(unpack_rect(rc)) > kKeepBits) {
          const uint32_t k = atomicAdd(&ls.nfull, 1u);
          ls.index[k] = (uint16_t)i;
          ls.first[k] = first;
          ls.org[k] = (uint32_t)rc;
          ls.end[k] = (uint32_t)(rc >> 32);
        }
      }
    }
    __syncthreads();
    if (TRAIN) {
      const uint32_t tx = (bx << bg.sx) + (uint32_t)(l & ((1 << bg.sx) - 1));
      const uint32_t ty = (by << bg.sy) + (uint32_t)((l & 31) >> bg.sx);
      for (uint32_t k = 2 * w + (l >> 5); k < ls.nfull; k += 2 * kLW) {
        const TileRect r = unpack_rect(ls.org[k] | ((uint64_t)ls.end[k] << 32));
        const uint32_t i = ls.index[k];
        if ((l & 31) < nt && tx >= r.x0 && tx < r.x1 && ty >= r.y0 && ty < r.y1 &&
            !((ls.mask[i] >> (l & 31)) & 1u)) {
          float2 *row = reinterpret_cast<float2 *>(
              ws.gpair + (size_t)kPairRow * (ls.first[k] + pair_rank(r, 0ull, tx, ty)));
#pragma unroll
          for (int q = 0; q < 4; ++q) row[q] = make_float2(0.0f, 0.0f);
          row[4] = make_float2(0.0f, __uint_as_float(ls.slot[i]));
        }
      }
    }
    for (uint32_t i0 = 0; i0 < cm; i0 += kWave) {
      const uint32_t i = min(i0 + (uint32_t)l, cm - 1u);
      const uint32_t s = ls.slot[i];
      const uint32_t bits = i0 + (uint32_t)l < cm ? ls.mask[i] : 0u;
#pragma unroll
      for (int q = 0; q < kTilesPerWave; ++q) {
        const bool hit = lt.on[q] && ((bits >> (w + q * kLW)) & 1u);
        const uint64_t hm = ballot(hit);
        if (hit) {
          const uint32_t dst = lt.run[q] + (uint32_t)__popcll(hm & lmask);
          ws.tkey[dst] = lt.tile[q];
          ws.tval[dst] = s;
        }
        lt.run[q] += (uint32_t)__popcll(hm);
      }
    }
  }
}

constexpr int kSliceBlocks = 256;  // blocks that write the lists of long bins

// The tile lists of one bin per block; those of long bins by the blocks from
// `slice0` on, a slice at a time, whose place in its tiles' lists is what the
// bin's earlier slices have counted; blocks from `order0` on: the compositing
// order (OCTGS_RASTER_TILE_ORDER).
template <bool TRAIN>
__global__ __launch_bounds__(kLT) void k_tile_lists(RasterWs ws, uint32_t slice0, uint32_t order0) {
  __shared__ union {
    ListSmem<TRAIN> ls;
    OrderSmem os;
  } sm;
  __shared__ uint32_t before[32];
  if (blockIdx.x >= order0) {
    order_tiles(ws, blockIdx.x - order0, sm.os);
    return;
  }
  const int t = threadIdx.x, w = t / kWave;
  const BinGrid &bg = ws.bins;
  const uint32_t nblk = TRAIN ? slot_blocks(ws.hdr->n_slots) : 1u;
  if (blockIdx.x < slice0) {
    const uint32_t nbins = (uint32_t)(bg.nx * bg.ny), bin = xcd_item(blockIdx.x, nbins);
    if (bin >= nbins) return;
    const uint2 rg = ws.bin_range[bin];
    if (rg.y == 0 || rg.y > (uint32_t)kBinCap) return;
    const uint32_t bx = bin % (uint32_t)bg.nx, by = bin / (uint32_t)bg.nx;
    ListTiles lt = list_tiles(ws, bx, by, w);
    append<TRAIN>(ws, sm.ls, lt, ws.bin_slot[0] + rg.x, ws.bin_mask[0] + rg.x, rg.y, bx, by, nblk);
    return;
  }
  const uint32_t ns = ws.hdr->n_slices;
  if (ns == 0u || ws.hdr->sync_error) return;
  for (uint32_t u = blockIdx.x - slice0; u < ns; u += order0 - slice0) {
    const uint32_t *row = ws.slices + kSliceRow * (size_t)u;
    const uint32_t bin = row[0], bx = bin % (uint32_t)bg.nx, by = bin / (uint32_t)bg.nx;
    const uint32_t at = ws.bin_range[bin].x + row[2];
    __syncthreads();  // the last slice's readers are done
    if (t < 32) before[t] = 0u;
    __syncthreads();
    // 16 slices at a time, a tile's count per thread
    uint32_t sum = 0;
    for (uint32_t i = (uint32_t)t / 32u; i < row[1]; i += kLT / 32)
      sum += row[(int64_t)(t % 32 + 4) - (int64_t)kSliceRow * (i + 1)];
    if (sum) atomicAdd(&before[t % 32], sum);
    __syncthreads();
    ListTiles lt = list_tiles(ws, bx, by, w);
#pragma unroll
    for (int q = 0; q < kTilesPerWave; ++q) lt.run[q] += before[w + q * kLW];
    append<TRAIN>(ws, sm.ls, lt, ws.bin_slot[1] + at, ws.bin_mask[1] + at, row[3], bx, by, nblk);
  }
}

}  // namespace

hipError_t launch_bin_sort(const RasterWs &ws, int band_row0, int rows, hipStream_t s) {
  const uint32_t nband = (uint32_t)(rows * ws.bins.nx);
  hipLaunchKernelGGL(k_bin_sort, dim3(xcd_blocks(nband)), dim3(kNT), 0, s, ws, band_row0, nband);
  if (rows < ws.bins.ny)
    hipLaunchKernelGGL(k_long_copy, dim3(kLongBlocks), dim3(kNT), 0, s, ws, band_row0, rows);
  return hipGetLastError();
}

hipError_t launch_tile_scan(const RasterWs &ws, bool train, hipStream_t s) {
  const int copied = ws.bins.band_rows < ws.bins.ny ? 1 : 0;
  hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)(ws.scan_blocks + 1 + kLongBlocks)),
                     dim3(kScanThreads), 0, s, ws, train ? 1 : 0, copied);
  return hipGetLastError();
}

hipError_t launch_tile_lists(const RasterWs &ws, bool train, bool ordered, hipStream_t s) {
  const uint32_t slice0 = xcd_blocks((uint32_t)(ws.bins.nx * ws.bins.ny));
  const uint32_t order0 = slice0 + kSliceBlocks;
  const dim3 grid(order0 + (ordered ? kXcds : 0u));
  if (train)
    hipLaunchKernelGGL(k_tile_lists<true>, grid, dim3(kLT), 0, s, ws, slice0, order0);
  else
    hipLaunchKernelGGL(k_tile_lists<false>, grid, dim3(kLT), 0, s, ws, slice0, order0);
  return hipGetLastError();
}

}  // namespace octgs
