// From grouped survivors to per-tile lists (the binning half of the forward
// rasterizer; Octree-GS Sec. III-A, tile-based front-to-back depth order).
//
// The projection leaves, per block of kSlots slots, the block's survivors
// grouped by screen bin.  Here:
//   k_bin_sort    one block per bin collects the bin's entries, sorts them by
//                 (depth bits, slot) in LDS, works out which of the bin's
//                 tiles each is listed in and counts the tiles' entries;
//   k_tile_scan   exclusive scan of the counts in tile order: each tile's
//                 range (and, in training, the blocks' pair numbers); its
//                 other blocks merge the sorted runs of bins whose list is
//                 longer than one block sorts at once;
//   k_tile_lists  one block per bin writes its tiles' lists in depth order:
//                 a wave takes a tile and compacts the bin's ordered entries
//                 by ballots, so all writes are in place and in order.
// No sort pass over pairs, no look-back chain over hundreds of partitions:
// the only waits on other blocks are the tile scan's (one block per 8,192
// tiles), bounded and on blocks that already run.
#include "octgs_internal.h"

namespace octgs {

namespace {

constexpr int kNT = kBinThreads, kNW = kNT / kWave;
constexpr int kDigit = 9, kDigits = 1 << kDigit;  // radix of the block sort: one digit per thread
constexpr int kSeg = 4, kRound = kSeg * kNT;      // slot blocks per thread and round of collect
static_assert(kDigits == kNT, "one digit per thread");

constexpr int kTestBatch = 256;  // long rectangles staged for their tile tests

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
  uint32_t vis, m, diff, flag, base, unknown;
};

// Index of the last of pre[0..kRound) that is <= i (pre[0] = 0, nondecreasing).
__device__ __forceinline__ uint32_t owner_of(const uint32_t *pre, uint32_t i) {
  uint32_t lo = 0;
#pragma unroll
  for (int st = kRound / 2; st > 0; st >>= 1)
    if (pre[lo + st] <= i) lo += st;
  return lo;
}

// All entries of a bin, in no particular order, handed to put(position, depth
// key, slot, tiles); returns their number.  local: the bin's index in its band.  On
// the first call (TOTALS) also the view's candidate and survivor counts into
// sm.cand and sm.vis.  Everything that one slot block says about the bin is
// loaded at once, then all entries and large survivors: two dependent round
// trips for up to 2,048 blocks.
template <bool TOTALS, typename Put>
__device__ __forceinline__ uint32_t collect(const RasterWs &ws, BinSmem &sm, int local, uint32_t bx,
                                            uint32_t by, uint32_t nblk, bool mine, Put put) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  if (t == 0) {
    sm.m = 0u;
    if (TOTALS) {
      sm.cand = 0ull;
      sm.vis = 0u;
    }
  }
  uint64_t cand = 0;
  uint32_t vis = 0;
  for (uint32_t r0 = 0; r0 < nblk; r0 += kRound) {
    uint32_t first[kSeg], c[kSeg], lc[kSeg], sc = 0, sl = 0;
#pragma unroll
    for (int j = 0; j < kSeg; ++j) {
      const uint32_t b = r0 + (uint32_t)(kSeg * t + j);
      const bool on = b < nblk;
      const uint32_t bc = on ? b : nblk - 1u;  // unconditional loads, all in flight together
      const uint16_t *row = ws.group_off + (size_t)bc * ws.group_pitch + local;
      const uint32_t e0 = row[0], e1 = row[1], lg = ws.blk_large[bc];
      if (TOTALS) {
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
    const uint32_t run = sm.m;
#pragma unroll
    for (int j = 0; j < kSeg; ++j) {
      sm.pre[kSeg * t + j] = es;
      sm.lpre[kSeg * t + j] = el;
      sm.first[kSeg * t + j] = (uint16_t)first[j];
      es += c[j];
      el += lc[j];
    }
    __syncthreads();
    if (t == 0) sm.m = run + ts;
    __syncthreads();
    for (uint32_t i0 = w * kWave; i0 < ts + tl; i0 += kNT) {
      const uint32_t i = i0 + l;
      const bool small = i < ts, large = !small && i < ts + tl;
      bool hit = false;
      uint4 e = make_uint4(0u, 0u, 0u, 0u);
      if (small) {
        const uint32_t o = owner_of(sm.pre, i);
        const uint4 v = ws.group[(size_t)(r0 + o) * kGroupCap + sm.first[o] + (i - sm.pre[o])];
        put(run + i, v.x, v.y, v.z);
      } else if (large) {
        const uint32_t o = owner_of(sm.lpre, i - ts);
        e = ws.large[(size_t)(r0 + o) * kSlots + (i - ts - sm.lpre[o])];
        const TileRect q = clip_to_bin(unpack_rect(e.x | ((uint64_t)e.y << 32)), ws.bins, bx, by);
        hit = q.x0 < q.x1 && q.y0 < q.y1;
      }
      const uint64_t hm = ballot(hit);
      if (hm == 0ull) continue;
      uint32_t p = 0;
      if (l == 0) p = atomicAdd(&sm.m, (uint32_t)__popcll(hm));
      p = (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
      if (hit) put(p + (uint32_t)__popcll(hm & lanemask_lt()), e.z, e.w, kTilesUnknown);
    }
    __syncthreads();
  }
  if (TOTALS) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) cand += __shfl_xor(cand, o, kWave);
    vis = wave_sum(vis);
    if (l == 0 && cand) atomicAdd(&sm.cand, (unsigned long long)cand);
    if (l == 0 && vis) atomicAdd(&sm.vis, vis);
  }
  __syncthreads();
  return sm.m;
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

// gkeys (nullable) receives the sorted keys.
template <int I>
__device__ __forceinline__ void sort_entries(BinSmem &sm, uint32_t m, uint32_t *gkeys) {
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
      if (gkeys)
        for (uint32_t i = t; i < m; i += kNT) gkeys[i] = sm.kk[i];
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

__device__ __forceinline__ void sort_any(BinSmem &sm, uint32_t m, uint32_t *gkeys) {
  static_assert(kBinItems == 8, "item counts of the sort");
  if (m <= kNT) sort_entries<1>(sm, m, gkeys);
  else if (m <= 2 * kNT) sort_entries<2>(sm, m, gkeys);
  else if (m <= 4 * kNT) sort_entries<4>(sm, m, gkeys);
  else sort_entries<8>(sm, m, gkeys);
}

// The tiles of the collected entries [0, cm) that came without them, and the
// number of entries per tile of the bin (lane j: tile j) of the wave's share.
// The unknown ones (long rectangles, up to a third of a bin and next to each
// other) are listed first (in sm.vv, unused until the sort); then half a wave
// takes an entry, a tile per lane, so that all lanes and waves share them.
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
  const uint32_t tx = (uint32_t)(l & ((1 << bg.sx) - 1)), ty = (uint32_t)((l & 31) >> bg.sx);
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
    for (uint32_t j = 2 * w; j < nk; j += 2 * kNW) {
      const uint32_t e = min(j + (uint32_t)(l >> 5), nk - 1u);
      const uint32_t box = sm.box[e];
      const bool in = tx >= (box & 15u) && tx < ((box >> 4) & 15u) && ty >= ((box >> 8) & 15u) &&
                      ty < ((box >> 12) & 15u);
      const bool hit = in && tile_meets_ellipse(sm.mx[e], sm.my[e], sm.qa[e], sm.qb[e], sm.qc[e],
                                                (bx << bg.sx) + tx, (by << bg.sy) + ty, ws.xmax,
                                                ws.ymax);
      const uint64_t hm = ballot(hit);
      if ((l & 31) == 0 && box != ~0u)
        sm.mm[sm.vv[k0 + e]] = l == 0 ? (uint32_t)hm : (uint32_t)(hm >> 32);
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
// on a 1920 x 1080 view of 862k pairs a block takes 22 us (collection 5.7,
// listing and testing long rectangles 6.3, counts 1.3, sort 6.3, writes 1.4) and
// the kernel 25; on 3840 x 2160 there are two rounds of blocks, 60.
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
  uint32_t m = collect<true>(ws, sm, local, bx, by, nblk, reach,
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
  if (over) m = 0;
  uint32_t mine = 0;
  if (m > 0) {
    // every entry stands for at least one candidate tile of its own, so the
    // lists of all bins fit the capacity
    uint32_t base = 0;
    const bool longer = m > (uint32_t)kBinCap;
    uint32_t *gkey = ws.tkey, *gslot = ws.bin_slot[0], *gmask = ws.bin_mask[0];
    if (longer) {
      // more than a block sorts at once: the entries to memory, then runs of
      // kBinCap, sorted one after the other; the tile scan merges them
      if (t == 0) {
        sm.base = atomicAdd(&ws.hdr->bin_cursor, m);
        ws.over_bin[atomicAdd(&ws.hdr->n_over, 1u)] = bin;
      }
      __syncthreads();
      const uint32_t gb = sm.base;
      collect<false>(ws, sm, local, bx, by, nblk, reach,
                     [&](uint32_t p, uint32_t key, uint32_t slot, uint32_t tiles) {
                       gkey[gb + p] = key;
                       gslot[gb + p] = slot;
                       gmask[gb + p] = tiles;
                     });
    }
    for (uint32_t c0 = 0; c0 < m; c0 += kBinCap) {
      const uint32_t cm = min((uint32_t)kBinCap, m - c0);
      if (longer) {
        __syncthreads();  // the last run's readers are done; the collected entries are written
        const uint32_t gb = sm.base;
        for (uint32_t i = t; i < cm; i += kNT) {
          sm.kk[i] = gkey[gb + c0 + i];
          sm.su[i] = gslot[gb + c0 + i];
          sm.mm[i] = gmask[gb + c0 + i];
        }
        __syncthreads();
      }
      mine += finish_tiles(ws, sm, cm, bx, by);
      // all bins ask at about the same time, and the answers come one after
      // the other: the sort, which loads nothing, covers the wait
      if (!longer && t == 0) base = atomicAdd(&ws.hdr->bin_cursor, m);
      sort_any(sm, cm, longer ? gkey + sm.base + c0 : nullptr);
      if (!longer && t == 0) sm.base = base;
      lds_barrier();
      const uint32_t gb = sm.base;
      for (uint32_t i = t; i < cm; i += kNT) {
        const uint32_t p = sm.vv[i] & ((1u << kPosBits) - 1u);
        gslot[gb + c0 + i] = sm.su[p];
        gmask[gb + c0 + i] = sm.mm[p];
      }
    }
    if (l < 32 && mine) atomicAdd(&sm.tcnt[l], mine);
    if (t == 0) ws.bin_range[bin] = make_uint2(sm.base, m);
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

// Entries of run r (entries [r0, r1) of a long list, sorted by (key, slot))
// that come before (k, s).
__device__ __forceinline__ uint32_t run_rank(const uint32_t *key, const uint32_t *slot, uint32_t r0,
                                             uint32_t r1, uint32_t k, uint32_t s) {
  uint32_t lo = r0, hi = r1;
  while (lo < hi) {
    const uint32_t mid = lo + (hi - lo) / 2;
    const uint32_t mk = key[mid];
    if (mk < k || (mk == k && slot[mid] < s)) lo = mid + 1;
    else hi = mid;
  }
  return lo - r0;
}

constexpr int kMergeBlocks = 128;

// Blocks [0, scan): ranges of kScanThreads * kScanTiles consecutive tiles each, chained
// by decoupled look-back; the block number is a ticket taken in the order
// blocks start, so every block that one waits on is already running.
// Block scan: pair numbers of the slot blocks (training).
// The others: entry by entry, the merge of long lists (an entry's place is its
// rank in its own run plus its ranks in the others).
__global__ __launch_bounds__(kScanThreads) void k_tile_scan(RasterWs ws, int train) {
  __shared__ uint32_t tmp[kScanThreads / kWave];
  __shared__ uint32_t s_b, s_excl;
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
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
      if (t0 + q >= ntiles) c[q] = 0u;
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
  if (blockIdx.x == (uint32_t)ws.scan_blocks) {
    if (!train) return;
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
    return;
  }
  // long lists: their entries, kScanThreads at a time, are dealt over the blocks
  __shared__ uint2 range[kScanThreads];
  __shared__ uint32_t chunk0[kScanThreads];
  const uint32_t nover = ws.hdr->n_over;
  const uint32_t mb = blockIdx.x - (uint32_t)ws.scan_blocks - 1u;
  const uint32_t *key = ws.tkey, *slot = ws.bin_slot[0];
  for (uint32_t q0 = 0; q0 < nover; q0 += kScanThreads) {
    const bool on = q0 + t < nover;
    const uint2 rt = on ? ws.bin_range[ws.over_bin[q0 + t]] : make_uint2(0u, 0u);
    uint32_t chunks;
    const uint32_t c0 = block_scan<kScanThreads>((rt.y + kScanThreads - 1) / kScanThreads, tmp, &chunks);
    range[t] = rt;
    chunk0[t] = c0;
    __syncthreads();
    for (uint32_t u = mb; u < chunks; u += kMergeBlocks) {
      uint32_t q = 0;  // the list of chunk u: the last that starts at or before it
#pragma unroll
      for (int st = kScanThreads / 2; st > 0; st >>= 1)
        if (q0 + q + st < nover && chunk0[q + st] <= u) q += st;
      const uint2 rg = range[q];
      const uint32_t i = (u - chunk0[q]) * kScanThreads + t;
      if (i >= rg.y) continue;
      const uint32_t own = i / kBinCap;
      const uint32_t k = key[rg.x + i], s = slot[rg.x + i];
      uint32_t rank = i - own * kBinCap;
      for (uint32_t c = 0; c * kBinCap < rg.y; ++c)
        if (c != own)
          rank += run_rank(key, slot, rg.x + c * kBinCap, rg.x + min((c + 1) * kBinCap, rg.y), k, s);
      ws.bin_slot[1][rg.x + rank] = s;
      ws.bin_mask[1][rg.x + rank] = ws.bin_mask[0][rg.x + i];
    }
    __syncthreads();  // before the next lists take their place
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

// The tile lists of one bin per block (blocks from `order0` on: the
// compositing order, OCTGS_RASTER_TILE_ORDER).  The bin's ordered entries are
// staged in LDS kLStage at a time; each wave walks them for up to four of the
// bin's tiles and appends those whose mask has the tile's bit.
// Training: rectangles with more than kKeepBits tiles number all their tiles
// as pairs; the rows of the numbers without a pair are cleared here, half a
// wave per entry, a tile per lane.
template <bool TRAIN>
__global__ __launch_bounds__(kLT) void k_tile_lists(RasterWs ws, uint32_t order0) {
  __shared__ union {
    ListSmem<TRAIN> ls;
    OrderSmem os;
  } sm;
  if (blockIdx.x >= order0) {
    order_tiles(ws, blockIdx.x - order0, sm.os);
    return;
  }
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const uint64_t lt = lanemask_lt();
  const BinGrid &bg = ws.bins;
  const uint32_t nbins = (uint32_t)(bg.nx * bg.ny), bin = xcd_item(blockIdx.x, nbins);
  if (bin >= nbins) return;
  const uint2 rg = ws.bin_range[bin];
  if (rg.y == 0) return;
  const uint32_t bx = bin % (uint32_t)bg.nx, by = bin / (uint32_t)bg.nx;
  const uint32_t nblk = TRAIN ? slot_blocks(ws.hdr->n_slots) : 1u;
  const int src = rg.y > (uint32_t)kBinCap;  // long lists are in the merged copy
  const uint32_t *slots = ws.bin_slot[src] + rg.x, *masks = ws.bin_mask[src] + rg.x;
  constexpr int kT = 32 / kLW;  // tiles per wave
  const int nt = 1 << (bg.sx + bg.sy);
  uint32_t tile[kT], run[kT];
  bool on[kT];
#pragma unroll
  for (int q = 0; q < kT; ++q) {
    const int j = w + q * kLW;
    const uint32_t tx = (bx << bg.sx) + (uint32_t)(j & ((1 << bg.sx) - 1));
    const uint32_t ty = (by << bg.sy) + (uint32_t)(j >> bg.sx);
    on[q] = j < nt && tx < (uint32_t)ws.tiles_x && ty < (uint32_t)ws.tiles_y;
    tile[q] = ty * (uint32_t)ws.tiles_x + tx;
    run[q] = on[q] ? ws.ranges[2 * (size_t)tile[q]] : 0u;
  }
  for (uint32_t c0 = 0; c0 < rg.y; c0 += kLStage) {
    const uint32_t cm = min((uint32_t)kLStage, rg.y - c0);
    __syncthreads();
    if (TRAIN) {
      if (t == 0) sm.ls.nfull = 0u;
      __syncthreads();
    }
    for (uint32_t i = t; i < cm; i += kLT) {
      const uint32_t s = slots[c0 + i];
      sm.ls.slot[i] = s;
      sm.ls.mask[i] = masks[c0 + i];
      if (TRAIN) {
        const uint64_t rc = ws.rect[s].x;
        const uint32_t first = ws.blk_pairs[slot_block(s, nblk)] + ws.pair_base[s];
        if (rect_tiles(unpack_rect(rc)) > kKeepBits) {
          const uint32_t k = atomicAdd(&sm.ls.nfull, 1u);
          sm.ls.index[k] = (uint16_t)i;
          sm.ls.first[k] = first;
          sm.ls.org[k] = (uint32_t)rc;
          sm.ls.end[k] = (uint32_t)(rc >> 32);
        }
      }
    }
    __syncthreads();
    if (TRAIN) {
      const uint32_t tx = (bx << bg.sx) + (uint32_t)(l & ((1 << bg.sx) - 1));
      const uint32_t ty = (by << bg.sy) + (uint32_t)((l & 31) >> bg.sx);
      for (uint32_t k = 2 * w + (l >> 5); k < sm.ls.nfull; k += 2 * kLW) {
        const TileRect r = unpack_rect(sm.ls.org[k] | ((uint64_t)sm.ls.end[k] << 32));
        const uint32_t i = sm.ls.index[k];
        if ((l & 31) < nt && tx >= r.x0 && tx < r.x1 && ty >= r.y0 && ty < r.y1 &&
            !((sm.ls.mask[i] >> (l & 31)) & 1u)) {
          float2 *row = reinterpret_cast<float2 *>(
              ws.gpair + (size_t)kPairRow * (sm.ls.first[k] + pair_rank(r, 0ull, tx, ty)));
#pragma unroll
          for (int q = 0; q < 4; ++q) row[q] = make_float2(0.0f, 0.0f);
          row[4] = make_float2(0.0f, __uint_as_float(sm.ls.slot[i]));
        }
      }
    }
    for (uint32_t i0 = 0; i0 < cm; i0 += kWave) {
      const uint32_t i = min(i0 + (uint32_t)l, cm - 1u);
      const uint32_t s = sm.ls.slot[i];
      const uint32_t bits = i0 + (uint32_t)l < cm ? sm.ls.mask[i] : 0u;
#pragma unroll
      for (int q = 0; q < kT; ++q) {
        const bool hit = on[q] && ((bits >> (w + q * kLW)) & 1u);
        const uint64_t hm = ballot(hit);
        if (hit) {
          const uint32_t dst = run[q] + (uint32_t)__popcll(hm & lt);
          ws.tkey[dst] = tile[q];
          ws.tval[dst] = s;
        }
        run[q] += (uint32_t)__popcll(hm);
      }
    }
  }
}

}  // namespace

hipError_t launch_bin_sort(const RasterWs &ws, int band_row0, int rows, hipStream_t s) {
  const uint32_t nband = (uint32_t)(rows * ws.bins.nx);
  hipLaunchKernelGGL(k_bin_sort, dim3(xcd_blocks(nband)), dim3(kNT), 0, s, ws, band_row0, nband);
  return hipGetLastError();
}

hipError_t launch_tile_scan(const RasterWs &ws, bool train, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)(ws.scan_blocks + 1 + kMergeBlocks)),
                     dim3(kScanThreads), 0, s, ws, train ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_tile_lists(const RasterWs &ws, bool train, bool ordered, hipStream_t s) {
  const uint32_t order0 = xcd_blocks((uint32_t)(ws.bins.nx * ws.bins.ny));
  const dim3 grid(order0 + (ordered ? kXcds : 0u));
  if (train)
    hipLaunchKernelGGL(k_tile_lists<true>, grid, dim3(kLT), 0, s, ws, order0);
  else
    hipLaunchKernelGGL(k_tile_lists<false>, grid, dim3(kLT), 0, s, ws, order0);
  return hipGetLastError();
}

}  // namespace octgs
