// From grouped survivors to per-tile lists (the binning half of the forward
// rasterizer; Octree-GS Sec. III-A, tile-based front-to-back depth order).
//
// The projection leaves, per block of kChunk slots, the block's survivors
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

struct BinSmem {
  uint32_t kk[kBinCap], ss[kBinCap];  // keys and slots being collected and sorted
  // wave digit counters of a sort pass; before, the starts of the blocks'
  // entries (one scan round) and their first positions
  union {
    uint16_t wcnt[kNW][256];
    struct {
      uint32_t pre[kNT];
      uint16_t first[kNT];
    };
  };
  uint32_t tmp[kNW];
  uint32_t tcnt[32];
  unsigned long long cand;
  uint32_t m, diff, flag, base;
};

// Index of the last of pre[0..kNT) that is <= i (pre[0] = 0, nondecreasing).
__device__ __forceinline__ uint32_t owner_of(const uint32_t *pre, uint32_t i) {
  uint32_t lo = 0;
#pragma unroll
  for (int st = kNT / 2; st > 0; st >>= 1)
    if (pre[lo + st] <= i) lo += st;
  return lo;
}

// All entries of a bin, in no particular order, handed to put(position, depth
// key, slot); returns their number.  local: the bin's index in its band.
template <typename Put>
__device__ __forceinline__ uint32_t collect(const RasterWs &ws, BinSmem &sm, int local, uint32_t bx,
                                            uint32_t by, uint32_t nblk, Put put) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const uint64_t lt = lanemask_lt();
  uint32_t run = 0, nlarge = 0;
  for (uint32_t r0 = 0; r0 < nblk; r0 += kNT) {
    const uint32_t b = r0 + t;
    uint32_t first = 0, c = 0;
    if (b < nblk) {
      const uint16_t *row = ws.group_off + (size_t)b * ws.group_pitch + local;
      first = row[0];
      c = row[1] - first;
      nlarge |= ws.blk_large[b];
    }
    uint32_t tot;
    const uint32_t ex = block_scan<kNT>(c, sm.tmp, &tot);
    sm.pre[t] = ex;
    sm.first[t] = (uint16_t)first;
    __syncthreads();
    for (uint32_t i = t; i < tot; i += kNT) {
      const uint32_t o = owner_of(sm.pre, i);
      const uint2 e = ws.group[(size_t)(r0 + o) * kGroupCap + sm.first[o] + (i - sm.pre[o])];
      put(run + i, e.x, e.y);
    }
    run += tot;
    __syncthreads();
  }
  if (t == 0) sm.m = run;
  if (__syncthreads_or((int)nlarge)) {
    for (uint32_t r0 = 0; r0 < nblk; r0 += kNT) {
      const uint32_t b = r0 + t;
      uint32_t tot;
      const uint32_t ex = block_scan<kNT>(b < nblk ? ws.blk_large[b] : 0u, sm.tmp, &tot);
      sm.pre[t] = ex;
      __syncthreads();
      for (uint32_t i0 = w * kWave; i0 < tot; i0 += kNT) {
        const uint32_t i = min(i0 + (uint32_t)l, tot - 1u);
        const uint32_t o = owner_of(sm.pre, i);
        const uint32_t slot = ws.large_slot[(size_t)(r0 + o) * kChunk + (i - sm.pre[o])];
        const ulonglong2 rm = ws.rect[slot];
        const TileRect r = unpack_rect(rm.x), c = clip_to_bin(r, ws.bins, bx, by);
        const bool hit = i0 + (uint32_t)l < tot && c.x0 < c.x1 && c.y0 < c.y1 &&
                         (rect_tiles(r) > kKeepBits || bin_tiles(r, rm.y, ws.bins, bx, by) != 0u);
        const uint64_t hm = ballot(hit);
        if (hm == 0ull) continue;
        uint32_t p = 0;
        if (l == 0) p = atomicAdd(&sm.m, (uint32_t)__popcll(hm));
        p = (uint32_t)__builtin_amdgcn_readfirstlane((int)p);
        if (hit) put(p + (uint32_t)__popcll(hm & lt), ws.depth[slot], slot);
      }
      __syncthreads();
    }
  }
  const uint32_t m = sm.m;
  __syncthreads();
  return m;
}

// Stable LSD radix sort of m keys (and one value each) held in registers,
// striped: item j of wave w is entry 64 (w I + j) + lane.  Only the digits in
// which `diff` has a bit are sorted.  Ends with the sorted keys and values in
// sm.kk and sm.ss.  Ranking is a match-any by ballots per item; each wave owns
// a contiguous run, so equal digits keep their order.
template <int I>
__device__ __forceinline__ void block_sort(BinSmem &sm, uint32_t (&key)[I], uint32_t (&val)[I],
                                           uint32_t m, uint32_t diff) {
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const uint64_t lt = lanemask_lt();
  const uint32_t e0 = (uint32_t)(w * I * kWave + l);
  bool placed = false;
  for (int shift = 0; shift < 32; shift += 8) {
    if (((diff >> shift) & 255u) == 0u) continue;
    __syncthreads();  // earlier readers of wcnt, kk and ss are done
    for (int i = t; i < kNW * 256 / 2; i += kNT) reinterpret_cast<uint32_t *>(sm.wcnt)[i] = 0u;
    __syncthreads();
    uint32_t rank[I];
#pragma unroll
    for (int j = 0; j < I; ++j) {
      const bool ok = e0 + (uint32_t)(j * kWave) < m;
      const uint32_t d = (key[j] >> shift) & 255u;
      uint64_t peers = ballot(ok);
#pragma unroll
      for (int b = 0; b < 8; ++b) {
        const int bit = (d >> b) & 1;
        const uint64_t bal = ballot(bit);
        peers &= bit ? bal : ~bal;
      }
      uint32_t before = 0;
      if (ok) before = sm.wcnt[w][d];
      // all lanes of the wave have read before any leader writes
      __builtin_amdgcn_wave_barrier();
      rank[j] = before + (uint32_t)__popcll(peers & lt);
      if (ok && (peers & lt) == 0ull) sm.wcnt[w][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // thread d < 256: the digit's count over the waves, then its start
    uint32_t tot = 0, all;
    if (t < 256) {
#pragma unroll
      for (int v = 0; v < kNW; ++v) {
        const uint32_t c = sm.wcnt[v][t];
        sm.wcnt[v][t] = (uint16_t)tot;
        tot += c;
      }
    }
    const uint32_t start = block_scan<kNT>(t < 256 ? tot : 0u, sm.tmp, &all);
    if (t < 256) {
#pragma unroll
      for (int v = 0; v < kNW; ++v) sm.wcnt[v][t] = (uint16_t)(sm.wcnt[v][t] + start);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < I; ++j) {
      if (e0 + (uint32_t)(j * kWave) < m) {
        const uint32_t pos = sm.wcnt[w][(key[j] >> shift) & 255u] + rank[j];
        sm.kk[pos] = key[j];
        sm.ss[pos] = val[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < I; ++j) {
      const uint32_t e = e0 + (uint32_t)(j * kWave);
      key[j] = e < m ? sm.kk[e] : 0u;
      val[j] = e < m ? sm.ss[e] : 0u;
    }
    placed = true;
  }
  if (!placed) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < I; ++j) {
      const uint32_t e = e0 + (uint32_t)(j * kWave);
      if (e < m) {
        sm.kk[e] = key[j];
        sm.ss[e] = val[j];
      }
    }
  }
  __syncthreads();
}

// OR over the block of the bits in which the keys differ from the first.
template <int I>
__device__ __forceinline__ uint32_t differing(BinSmem &sm, const uint32_t (&key)[I], uint32_t first,
                                              uint32_t m) {
  const uint32_t e0 = (uint32_t)(threadIdx.x / kWave * I * kWave + __lane_id());
  uint32_t d = 0;
#pragma unroll
  for (int j = 0; j < I; ++j)
    if (e0 + (uint32_t)(j * kWave) < m) d |= key[j] ^ first;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) d |= (uint32_t)__shfl_xor((int)d, o, kWave);
  if (threadIdx.x == 0) sm.diff = 0u;
  __syncthreads();
  if (__lane_id() == 0 && d) atomicOr(&sm.diff, d);
  __syncthreads();
  return sm.diff;
}

// Sorts the m entries of sm.kk / sm.ss by (key, slot).  Entries arrive in no
// order, so equal keys (a few per bin: depths are floats) are put into slot
// order afterwards: short runs by the thread that owns the run's head, and
// where a run is longer than kRun all entries are sorted again, by slot first.
constexpr uint32_t kRun = 16;

template <int I>
__device__ __forceinline__ void sort_entries(BinSmem &sm, uint32_t m) {
  const int t = threadIdx.x;
  const uint32_t e0 = (uint32_t)(t / kWave * I * kWave + __lane_id());
  uint32_t key[I], val[I];
#pragma unroll
  for (int j = 0; j < I; ++j) {
    const uint32_t e = e0 + (uint32_t)(j * kWave);
    key[j] = e < m ? sm.kk[e] : 0u;
    val[j] = e < m ? sm.ss[e] : 0u;
  }
  const uint32_t diff = differing<I>(sm, key, sm.kk[0], m);
  block_sort<I>(sm, key, val, m, diff);
  if (t == 0) sm.flag = 0u;
  __syncthreads();
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
      const uint32_t v = sm.ss[a];
      uint32_t b = a;
      for (; b > i && sm.ss[b - 1] > v; --b) sm.ss[b] = sm.ss[b - 1];
      sm.ss[b] = v;
    }
  }
  __syncthreads();
  if (sm.flag) {
#pragma unroll
    for (int j = 0; j < I; ++j) {
      const uint32_t e = e0 + (uint32_t)(j * kWave);
      key[j] = e < m ? sm.kk[e] : 0u;
      val[j] = e < m ? sm.ss[e] : 0u;
    }
    const uint32_t sd = differing<I>(sm, val, sm.ss[0], m);
    block_sort<I>(sm, val, key, m, sd);  // leaves the slots in kk and the keys in ss
#pragma unroll
    for (int j = 0; j < I; ++j) {
      const uint32_t e = e0 + (uint32_t)(j * kWave);
      val[j] = e < m ? sm.kk[e] : 0u;
      key[j] = e < m ? sm.ss[e] : 0u;
    }
    block_sort<I>(sm, key, val, m, diff);
  }
}

__device__ __forceinline__ void sort_any(BinSmem &sm, uint32_t m) {
  static_assert(kBinItems == 8, "item counts of the sort");
  if (m <= kNT) sort_entries<1>(sm, m);
  else if (m <= 2 * kNT) sort_entries<2>(sm, m);
  else if (m <= 4 * kNT) sort_entries<4>(sm, m);
  else sort_entries<8>(sm, m);
}

// Tiles of bin (bx, by) in which slot is listed: from its keep mask, or, for
// a rectangle with more tiles than that holds, by the tile test here.
__device__ __forceinline__ uint32_t entry_tiles(const RasterWs &ws, uint32_t slot, uint32_t bx,
                                                uint32_t by) {
  const ulonglong2 rm = ws.rect[slot];
  const TileRect r = unpack_rect(rm.x);
  if (rect_tiles(r) <= kKeepBits) return bin_tiles(r, rm.y, ws.bins, bx, by);
  const TileRect c = clip_to_bin(r, ws.bins, bx, by);
  const float4 A = ws.proj[3 * (size_t)slot], Q = ws.proj[3 * (size_t)slot + 2];
  uint32_t bits = 0;
  for (uint32_t ty = c.y0; ty < c.y1; ++ty)
    for (uint32_t tx = c.x0; tx < c.x1; ++tx)
      if (tile_meets_ellipse(A.x, A.y, Q.y, Q.z, Q.w, tx, ty, ws.xmax, ws.ymax))
        bits |= 1u << (((ty - (by << ws.bins.sy)) << ws.bins.sx) + (tx - (bx << ws.bins.sx)));
  return bits;
}

// One block per bin of the band.  Bound by latency: a chain of about 25
// barriers and LDS round trips for lists of up to 1,024 entries (three or four
// digit passes), with one block of 16 waves per bin and up to two per compute
// unit.
__global__ __launch_bounds__(kNT) void k_bin_sort(RasterWs ws, int band_row0) {
  __shared__ BinSmem sm;
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  const BinGrid &bg = ws.bins;
  const uint32_t bx = blockIdx.x % (uint32_t)bg.nx;
  const uint32_t by = (uint32_t)band_row0 + blockIdx.x / (uint32_t)bg.nx;
  const uint32_t bin = by * (uint32_t)bg.nx + bx;
  const uint32_t nblk = (ws.hdr->n_slots + kChunk - 1) / kChunk;
  if (t == 0) {
    sm.cand = 0ull;
    sm.flag = 0u;
  }
  if (t < 32) sm.tcnt[t] = 0u;
  __syncthreads();
  // candidates of the whole view: nothing is listed if they exceed the capacity
  {
    uint64_t c = 0;
    uint32_t v = 0;
    for (uint32_t b = t; b < nblk; b += kNT) {
      c += ws.blk_cand[b];
      if (bin == 0) v += ws.blk_vis[b];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
    if (l == 0 && c) atomicAdd(&sm.cand, (unsigned long long)c);
    if (bin == 0) {
      v = wave_sum(v);
      if (l == 0 && v) atomicAdd(&sm.flag, v);
    }
  }
  __syncthreads();
  const uint32_t cand = (uint32_t)std::min<uint64_t>(sm.cand, kLbVal);
  const bool over = cand > (uint64_t)ws.pcap;
  if (bin == 0 && t == 0) {
    ws.hdr->n_visible = sm.flag;
    ws.hdr->n_candidates = cand;
    ws.hdr->pair_overflow = over ? 1u : 0u;
  }
  uint32_t m = 0;
  const int local = (int)((by - (uint32_t)band_row0) * (uint32_t)bg.gx + bx);
  if (!over && bx < (uint32_t)bg.gx)
    m = collect(ws, sm, local, bx, by, nblk, [&](uint32_t p, uint32_t key, uint32_t slot) {
      if (p < (uint32_t)kBinCap) {
        sm.kk[p] = key;
        sm.ss[p] = slot;
      }
    });
  uint32_t mine = 0;  // lane j < 32: entries of the bin's tile j in this wave's share
  if (m > 0) {
    // every entry stands for at least one candidate tile of its own, so the
    // lists of all bins fit the capacity
    if (t == 0) sm.base = atomicAdd(&ws.hdr->bin_cursor, m);
    __syncthreads();
    const uint32_t base = sm.base;
    const bool longer = m > (uint32_t)kBinCap;
    uint32_t *gkey = ws.tkey, *gslot = ws.bin_slot[0];
    if (longer) {
      // more than a block sorts at once: the entries to memory, then runs of
      // kBinCap, sorted one after the other; the tile scan merges them
      collect(ws, sm, local, bx, by, nblk,
              [&](uint32_t p, uint32_t key, uint32_t slot) {
                gkey[base + p] = key;
                gslot[base + p] = slot;
              });
      if (t == 0) ws.over_bin[atomicAdd(&ws.hdr->n_over, 1u)] = bin;
    }
    for (uint32_t c0 = 0; c0 < m; c0 += kBinCap) {
      const uint32_t cm = min((uint32_t)kBinCap, m - c0);
      if (longer) {
        __syncthreads();  // the last run's readers are done; the collected entries are written
        for (uint32_t i = t; i < cm; i += kNT) {
          sm.kk[i] = gkey[base + c0 + i];
          sm.ss[i] = gslot[base + c0 + i];
        }
        __syncthreads();
      }
      sort_any(sm, cm);
      __syncthreads();
      for (uint32_t i0 = w * kWave; i0 < cm; i0 += kNT) {
        const uint32_t i = i0 + l;
        uint32_t bits = 0;
        if (i < cm) {
          const uint32_t slot = sm.ss[i];
          bits = entry_tiles(ws, slot, bx, by);
          gslot[base + c0 + i] = slot;
          ws.bin_mask[0][base + c0 + i] = bits;
          if (longer) gkey[base + c0 + i] = sm.kk[i];
        }
        const int nt = 1 << (bg.sx + bg.sy);
        for (int j = 0; j < nt; ++j) {
          const uint32_t c = (uint32_t)__popcll(ballot((bits >> j) & 1u));
          if (l == j) mine += c;
        }
      }
    }
    if (l < 32 && mine) atomicAdd(&sm.tcnt[l], mine);
    if (t == 0) ws.bin_range[bin] = make_uint2(base, m);
  } else if (t == 0) {
    ws.bin_range[bin] = make_uint2(0u, 0u);
  }
  __syncthreads();
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

// Blocks [0, scan): ranges of kNT * kScanTiles consecutive tiles each, chained
// by decoupled look-back; the block number is a ticket taken in the order
// blocks start, so every block that one waits on is already running.
// Block scan: pair numbers of the slot blocks (training).
// The others: entry by entry, the merge of long lists (an entry's place is its
// rank in its own run plus its ranks in the others).
__global__ __launch_bounds__(kNT) void k_tile_scan(RasterWs ws, int train) {
  __shared__ uint32_t tmp[kNW];
  __shared__ uint32_t s_b, s_excl;
  const int t = threadIdx.x, w = t / kWave, l = __lane_id();
  if (blockIdx.x < (uint32_t)ws.scan_blocks) {
    if (t == 0) s_b = ws.scan_blocks > 1 ? atomicAdd(&ws.hdr->scan_ticket, 1u) : 0u;
    __syncthreads();
    const uint32_t b = s_b;
    const int64_t ntiles = (int64_t)ws.tiles_x * ws.tiles_y;
    const int64_t t0 = ((int64_t)b * kNT + t) * kScanTiles;
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
    uint32_t run = block_scan<kNT>(sum, tmp, &tot);
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
      if (t0 + q < ntiles) out[q] = make_uint2(run, run + c[q]);
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
    const uint32_t nblk = (ws.hdr->n_slots + kChunk - 1) / kChunk;
    uint32_t run = 0;
    for (uint32_t r0 = 0; r0 < nblk; r0 += kNT) {
      const uint32_t b = r0 + t;
      uint32_t tot;
      const uint32_t ex = block_scan<kNT>(b < nblk ? ws.blk_pairs[b] : 0u, tmp, &tot);
      if (b < nblk) ws.blk_pairs[b] = run + ex;
      run += tot;
    }
    if (t == 0) ws.hdr->n_emit = ws.hdr->pair_overflow ? 0u : run;
    return;
  }
  const uint32_t nover = ws.hdr->n_over;
  const uint32_t mb = blockIdx.x - (uint32_t)ws.scan_blocks - 1u;
  const uint32_t *key = ws.tkey, *slot = ws.bin_slot[0];
  for (uint32_t q = 0; q < nover; ++q) {
    const uint2 rg = ws.bin_range[ws.over_bin[q]];
    for (uint32_t i = mb * kNT + t; i < rg.y; i += kMergeBlocks * kNT) {
      const uint32_t own = i / kBinCap;
      const uint32_t k = key[rg.x + i], s = slot[rg.x + i];
      uint32_t rank = i - own * kBinCap;
      for (uint32_t c = 0; c * kBinCap < rg.y; ++c)
        if (c != own)
          rank += run_rank(key, slot, rg.x + c * kBinCap, rg.x + min((c + 1) * kBinCap, rg.y), k, s);
      ws.bin_slot[1][rg.x + rank] = s;
      ws.bin_mask[1][rg.x + rank] = ws.bin_mask[0][rg.x + i];
    }
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
  uint64_t keep[TRAIN ? kLStage : 1];
  uint32_t first[TRAIN ? kLStage : 1], xy[TRAIN ? kLStage : 1], wd[TRAIN ? kLStage : 1];
};
constexpr uint32_t kHuge = 1u << 31;

// The tile lists of one bin per block (blocks from `order0` on: the
// compositing order, OCTGS_RASTER_TILE_ORDER).  The bin's ordered entries are
// staged in LDS kLStage at a time; each wave walks them for up to four of the
// bin's tiles and appends those whose mask has the tile's bit.
// Training: each pair also gets its pair number, the slot's first number plus
// the tile's rank among the kept tiles of the rectangle (row-major), so that a
// Gaussian's numbers are contiguous; rectangles with more than kKeepBits tiles
// number all their tiles, and the rows of the numbers without a pair are
// cleared here.
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
  const uint32_t bin = blockIdx.x;
  const uint2 rg = ws.bin_range[bin];
  if (rg.y == 0) return;
  const uint32_t bx = bin % (uint32_t)bg.nx, by = bin / (uint32_t)bg.nx;
  const int src = rg.y > (uint32_t)kBinCap;  // long lists are in the merged copy
  const uint32_t *slots = ws.bin_slot[src] + rg.x, *masks = ws.bin_mask[src] + rg.x;
  constexpr int kT = 32 / kLW;  // tiles per wave
  const int nt = 1 << (bg.sx + bg.sy);
  uint32_t tile[kT], tx[kT], ty[kT], run[kT];
  bool on[kT];
#pragma unroll
  for (int q = 0; q < kT; ++q) {
    const int j = w + q * kLW;
    tx[q] = (bx << bg.sx) + (uint32_t)(j & ((1 << bg.sx) - 1));
    ty[q] = (by << bg.sy) + (uint32_t)(j >> bg.sx);
    on[q] = j < nt && tx[q] < (uint32_t)ws.tiles_x && ty[q] < (uint32_t)ws.tiles_y;
    tile[q] = ty[q] * (uint32_t)ws.tiles_x + tx[q];
    run[q] = on[q] ? ws.ranges[2 * (size_t)tile[q]] : 0u;
  }
  for (uint32_t c0 = 0; c0 < rg.y; c0 += kLStage) {
    const uint32_t cm = min((uint32_t)kLStage, rg.y - c0);
    __syncthreads();
    for (uint32_t i = t; i < cm; i += kLT) {
      const uint32_t s = slots[c0 + i];
      sm.ls.slot[i] = s;
      sm.ls.mask[i] = masks[c0 + i];
      if (TRAIN) {
        const ulonglong2 rm = ws.rect[s];
        const TileRect r = unpack_rect(rm.x);
        sm.ls.keep[i] = rm.y;
        sm.ls.first[i] = ws.blk_pairs[s / kChunk] + ws.pair_base[s];
        sm.ls.xy[i] = r.x0 | (r.y0 << 16);
        sm.ls.wd[i] = (r.x1 - r.x0) | (rect_tiles(r) > kKeepBits ? kHuge : 0u);
      }
    }
    __syncthreads();
    for (uint32_t i0 = 0; i0 < cm; i0 += kWave) {
      const uint32_t i = min(i0 + (uint32_t)l, cm - 1u);
      const uint32_t s = sm.ls.slot[i];
      const uint32_t bits = i0 + (uint32_t)l < cm ? sm.ls.mask[i] : 0u;
#pragma unroll
      for (int q = 0; q < kT; ++q) {
        const bool hit = on[q] && ((bits >> (w + q * kLW)) & 1u);
        const uint64_t hm = ballot(hit);
        const uint32_t dst = run[q] + (uint32_t)__popcll(hm & lt);
        run[q] += (uint32_t)__popcll(hm);
        if (hit) {
          ws.tkey[dst] = tile[q];
          ws.tval[dst] = s;
        }
        if (TRAIN && on[q] && i0 + (uint32_t)l < cm) {
          const uint32_t xy = sm.ls.xy[i], wd = sm.ls.wd[i], wid = wd & ~kHuge;
          const uint32_t rx = tx[q] - (xy & 0xffffu), ry = ty[q] - (xy >> 16);
          const uint32_t loc = ry * wid + rx, first = sm.ls.first[i];
          if (hit)
            ws.tpair[dst] = first + ((wd & kHuge) ? loc
                                                  : (uint32_t)__popcll(sm.ls.keep[i] & ((1ull << (loc & 63u)) - 1ull)));
          if ((wd & kHuge) && !hit) {
            // a number without a pair, if the tile lies in the rectangle
            const TileRect r = unpack_rect(ws.rect[s].x);
            if (tx[q] >= r.x0 && tx[q] < r.x1 && ty[q] >= r.y0 && ty[q] < r.y1) {
              float *row = ws.gpair + (size_t)kPairRow * (first + loc);
#pragma unroll
              for (int k = 0; k < 9; ++k) row[k] = 0.0f;
              row[9] = __uint_as_float(s);
            }
          }
        }
      }
    }
  }
}

}  // namespace

hipError_t launch_bin_sort(const RasterWs &ws, int band_row0, int rows, hipStream_t s) {
  hipLaunchKernelGGL(k_bin_sort, dim3((unsigned)(rows * ws.bins.nx)), dim3(kNT), 0, s, ws, band_row0);
  return hipGetLastError();
}

hipError_t launch_tile_scan(const RasterWs &ws, bool train, hipStream_t s) {
  hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)(ws.scan_blocks + 1 + kMergeBlocks)), dim3(kNT), 0,
                     s, ws, train ? 1 : 0);
  return hipGetLastError();
}

hipError_t launch_tile_lists(const RasterWs &ws, bool train, bool ordered, hipStream_t s) {
  const uint32_t nbins = (uint32_t)(ws.bins.nx * ws.bins.ny);
  const dim3 grid(nbins + (ordered ? kXcds : 0u));
  if (train)
    hipLaunchKernelGGL(k_tile_lists<true>, grid, dim3(kLT), 0, s, ws, nbins);
  else
    hipLaunchKernelGGL(k_tile_lists<false>, grid, dim3(kLT), 0, s, ws, nbins);
  return hipGetLastError();
}

}  // namespace octgs
