// Work items of the forward and of the dQ kernel, built on the device by one
// workgroup.
#pragma once

#include "attn_common.h"

namespace libra {

// Work items: every tile is split into sample fragments; every fragment into
// items of (<= 4 heads of one KV group) x (32 * 4 / heads rows), starting at
// the fragment's first row.  The enumeration goes by 32-row windows of a tile:
// f(item, key blocks) is called for the items whose first row lies in rows
// [wa, wb) of tile t (wb - wa <= 32, so at most one item per fragment and
// head chunk), which spreads a tile's items over many threads.
template <typename F>
__device__ void for_each_fwd_item_in(const libra_tile_t &t, int64_t wa, int64_t wb,
                                     const CuView &cu, int64_t n, int G, F &&f) {
  int64_t j = upper_bound64(cu, n, wa) - 1;
  for (; j < n && cu[j] < wb; ++j) {
    const int64_t pb = t.q_begin > cu[j] ? t.q_begin : cu[j];
    const int64_t pe = t.q_end < cu[j + 1] ? t.q_end : cu[j + 1];
    const int32_t row0 = (int32_t)(t.q_row + (pb - t.q_begin));
    const int32_t qloc0 = (int32_t)(pb - cu[j]);
    const int32_t nfrag = (int32_t)(pe - pb);
    const int64_t lim = wb < pe ? wb : pe;
    for (int g = t.head_begin / G; g * G < t.head_end; ++g) {
      const int hl = max(t.head_begin, g * G), hh = min(t.head_end, (g + 1) * G);
      for (int h0 = hl; h0 < hh; h0 += 4) {
        const int nh = min(4, hh - h0);
        const int rows_per = kRows * (4 / nh);
        // first item start pb + k rows_per at or after wa
        int64_t k = wa > pb ? (wa - pb + rows_per - 1) / rows_per : 0;
        for (; pb + k * rows_per < lim; ++k) {
          const int32_t rb = (int32_t)(k * rows_per);
          const int nrows = min(rows_per, nfrag - rb);
          const int32_t nkb = (qloc0 + rb + nrows - 1) / kFwdBN + 1;
          FwdItem it{row0 + rb, qloc0 + rb, (int32_t)j, h0, nh, nrows, g, 0, nkb, -1, 0, 0};
          f(it, nkb);
        }
      }
    }
  }
}

// One workgroup: every tile's items, longest-first, one queue per XCD keyed
// by (KV head, head chunk) so that an XCD streams few K/V sequences.  Tiles
// outside the buffers are skipped, and counted in hdr[kBadTiles] when
// `count_bad` is set.  The backward counts them in the dK / dV part of its
// preparation, which runs beside this one and zeroes that slot, so an overflow of
// this list goes to a slot of its own there (hdr[kDqFull]).
//
// Split K: when there are fewer than two items per workgroup of `split_grid`
// (few rows and heads against long samples), and with
// `idle_only` only when whole rounds of that many items would leave more than a
// tenth of the workgroups idle, the key blocks that all rows of an item
// attend in full (below its first row's block kd) are cut into ranges of C
// blocks, about four items per workgroup in all;
// the last range also takes the blocks from kd on, so that every row has a
// key in the first block of every range.  Items with kd < 2 C stay whole.
// Each part writes a partial result to its own slot (max_parts slots;
// max_parts = 0 never splits) and fwd_combine_kernel merges the parts of
// every split item.  C is at least kFwdSplitMinBlocks and doubles until the
// parts fit the slots.
struct FwdPrep {
  const int64_t *cu;
  int64_t n;
  const libra_tile_t *tiles;
  int64_t T;
  int h_q, h_kv;
  int64_t n_q, n_kv;
  int32_t *hdr;
  FwdItem *items;
  int64_t max_items;
  int count_bad;
  int grid;        // workgroups that run the items
  int split_grid;  // workgroups that the split rule counts
  int max_parts, idle_only;
  FwdSplit *splits;
};
struct FwdPrepLds {
  int32_t hist[kXcds * kQBuckets];
  int32_t part[kPrepThreads];
  int32_t cu[kCuLds];
  unsigned long long wmax, items, work, parts, pairs;
  int32_t chunk, nslot, nsplit;
};
__device__ __forceinline__ void prep_fwd(const FwdPrep &a, FwdPrepLds &lds) {
  const int64_t n = a.n, T = a.T, n_q = a.n_q, n_kv = a.n_kv;
  const libra_tile_t *tiles = a.tiles;
  const int h_q = a.h_q, h_kv = a.h_kv, grid = a.split_grid, max_parts = a.max_parts;
  int32_t *hdr = a.hdr;
  auto &s_wmax = lds.wmax, &s_items = lds.items, &s_work = lds.work, &s_parts = lds.parts,
       &s_pairs = lds.pairs;
  auto &s_chunk = lds.chunk, &s_nslot = lds.nslot, &s_nsplit = lds.nsplit;
  const CuView cu = cu_view(a.cu, n, lds.cu);
  const int tid = threadIdx.x;
  const int G = h_q / h_kv;
  const int chunks = (G + 3) / 4;                    // head chunks per KV group
  const int keys = h_kv * chunks;
  const int R = keys >= kXcds ? 1 : kXcds / keys;    // queues per key
  if (tid == 0) {
    hdr[a.count_bad ? kBadTiles : kDqFull] = 0;
    hdr[kFwdSplits] = 0;
    hdr[kFwdSplits + 1] = 0;
    s_wmax = 0;
    s_pairs = 0;
    s_items = 0;
    s_work = 0;
    s_chunk = 0;
    s_nslot = 0;
    s_nsplit = 0;
  }
  __threadfence();
  __syncthreads();
  // bad tiles, and the 32-row windows of the longest good tile
  int bad = 0;
  unsigned long long wm = 0, pairs = 0;
  for (int64_t t = tid; t < T; t += kPrepThreads) {
    const libra_tile_t tl = tiles[t];
    if (!tile_ok(tl, n_q, n_kv, h_q)) {
      ++bad;
      continue;
    }
    const unsigned long long w = (unsigned long long)((tl.q_end - tl.q_begin + kRows - 1) / kRows);
    wm = w > wm ? w : wm;
    pairs += (unsigned long long)(tl.q_end - tl.q_begin) * (unsigned long long)(tl.head_end - tl.head_begin);
  }
  if (bad && a.count_bad) atomicAdd(&hdr[kBadTiles], bad);
  if (wm) atomicMax(&s_wmax, wm);
  if (pairs) atomicAdd(&s_pairs, pairs);
  __syncthreads();
  const int64_t wmax = (int64_t)s_wmax;
  // every whole item once: f(item, queue)
  auto whole = [&](auto &&f) {
    for (int64_t v = tid; v < T * wmax; v += kPrepThreads) {
      const bool small = T * wmax < INT32_MAX;   // a 32-bit division, not a 64-bit one
      const int64_t t = small ? (int64_t)((uint32_t)v / (uint32_t)wmax) : v / wmax;
      const int64_t w = v - t * wmax;
      const libra_tile_t tl = tiles[t];
      if (!tile_ok(tl, n_q, n_kv, h_q)) continue;
      const int64_t wa = tl.q_begin + (int64_t)kRows * w;
      if (wa >= tl.q_end) continue;
      const int64_t wb = wa + kRows < tl.q_end ? wa + kRows : tl.q_end;
      for_each_fwd_item_in(tl, wa, wb, cu, n, G, [&](const FwdItem &it, int) {
        const int key = it.g * chunks + (it.head0 - it.g * G) / 4;
        f(it, (key * R + (it.q_row0 / 128) % R) % kXcds);
      });
    }
  };
  // an item covers at most 128 (row, head) pairs: with pairs / 128 items or
  // more there are enough for the grid, and the item count is not needed
  if (max_parts > 0 && s_pairs / 128 < 2ull * (unsigned long long)grid) {
    whole([&](const FwdItem &it, int) {
      atomicAdd(&s_items, 1ull);
      atomicAdd(&s_work, (unsigned long long)it.kb1);
    });
    __syncthreads();
    const unsigned long long n_items = s_items, work = s_work, gr = (unsigned long long)grid;
    // rounds of that many items fill less than 90% of the workgroups
    const bool idle = n_items * 10 < (n_items + gr - 1) / gr * gr * 9;
    if (n_items > 0 && n_items < 2 * gr && (idle || !a.idle_only)) {
      long long c = (long long)((work + 4ull * grid - 1) / (4ull * grid));
      c = c > kFwdSplitMinBlocks ? c : kFwdSplitMinBlocks;
      for (; c < (1ll << 30); c *= 2) {   // at most ~30 rounds; the first fits by construction
        if (tid == 0) s_parts = 0;
        __syncthreads();
        whole([&](const FwdItem &it, int) {
          const long long np = (it.q_loc0 / kFwdBN) / c;
          if (np >= 2) atomicAdd(&s_parts, (unsigned long long)np);
        });
        __syncthreads();
        const bool fits = s_parts <= (unsigned long long)max_parts;
        __syncthreads();
        if (fits) break;
      }
      if (tid == 0) s_chunk = (int32_t)(c < (1ll << 30) ? c : 0);
    }
    __syncthreads();
  }
  const int chunk = s_chunk;   // 0: no item is split
  auto each = [&](auto &&f, bool scatter) {
    whole([&](const FwdItem &it, int x) {
      const int np = chunk ? (it.q_loc0 / kFwdBN) / chunk : 0;
      if (np < 2) {
        f(it, (int64_t)it.kb1, x);
        return;
      }
      int32_t base = 0;
      if (scatter) {
        base = atomicAdd(&s_nslot, np);
        a.splits[atomicAdd(&s_nsplit, 1)] = FwdSplit{it, base, np, 0, 0};
      }
      for (int p = 0; p < np; ++p) {
        FwdItem ip = it;
        ip.kb0 = p * chunk;
        ip.kb1 = p + 1 < np ? (p + 1) * chunk : it.kb1;
        ip.slot = base + p;
        f(ip, (int64_t)(ip.kb1 - ip.kb0), x);
      }
    });
  };
  build_queues<FwdItem>(each, lds.hist, lds.part, hdr, kFwdQ,
                        a.count_bad ? kBadTiles : kDqFull, a.items, a.max_items, a.grid);
  __syncthreads();
  if (tid == 0) {
    hdr[kFwdSplits] = s_nsplit;
    hdr[kFwdSplits + 1] = s_nslot;
  }
}

}  // namespace libra
