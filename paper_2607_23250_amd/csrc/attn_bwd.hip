// Backward pass of document-masked causal attention over SH-Tiles (gfx950).
//
// Textbook attention gradients (the paper's backward reuses the forward
// assignment with reversed transfers, Sec. 4.3.3, so it computes exactly
// these): P = exp(S - LSE), D = rowsum(dO * O), dV = P^T dO,
// dS = P * (dO V^T - D), dQ = scale dS K, dK = scale dS^T Q.
//
// Two persistent kernels, no atomics (every output element has one writer):
//   * dK / dV (here), KV-stationary: a work item is 128 keys of one KV head of
//     one sample (anchored at the sample start); each of the 4 waves keeps 32
//     keys of K and V in registers plus fp32 dK^T / dV^T accumulators and
//     loops over the 32-row query blocks of the tiles that attend them, two
//     query heads of the KV group per step.  S and dP are computed with
//     queries on M (lane = key), exactly the operand layout that dV^T = dO^T P
//     and dK^T = Q^T dS need; the dO^T / Q^T operands come from the same LDS
//     tiles through the LDS transpose reads.  LSE and D enter the S and dP
//     products as one extra k-block (see pre_pass), so the VALU only
//     exponentiates and multiplies.  A step's Q, dO and extra operands are two
//     contiguous records that the pre-pass lays out as the LDS stage wants
//     them; steps are staged in a 4-deep LDS ring, three ahead of the one
//     computed.
//     One wave per SIMD issues everything, so the kernel is bound by its
//     instruction stream and by the products (1.30 PFLOP/s of them on the
//     256K share, against 1.56 of a large matrix product).  dK / dV on the
//     256K share, same box: row-major copies 98.9 ms (about 850 instructions
//     per step, 66 of them address additions, 58 spilled scalars); records
//     93.3; the copies posted between the product phases instead of at the top
//     91.4 to 92.9; the two heads of a step pipelined against one another
//     (about 490 instructions) 3% less again.
//   * dQ (attn_bwd_dq.hip), query-stationary, shaped like the forward.  It
//     recomputes S and dP instead of accumulating dQ across key blocks with
//     atomics: on long samples that accumulation is read-modify-write traffic
//     of 4 bytes x d per (32 queries x 128 keys) per head, which would bound
//     the whole backward by HBM.
// Preparation: D = rowsum(dO * O), the augmented operands and the two
// work-item lists, longest first.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "attn_common.h"
#include "attn_items.h"
#include "errors.h"

namespace libra {

__device__ __forceinline__ unsigned long long ld_agent(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Bit set of the KV heads whose query groups intersect [hb, he); `odd` is set
// if it covers an odd number of heads of one of them.
__device__ __forceinline__ unsigned long long group_bits(int hb, int he, int G, bool &odd) {
  unsigned long long m = 0;
  for (int g = hb / G; g * G < he; ++g) {
    m |= 1ull << g;
    odd |= ((min(he, (g + 1) * G) - max(hb, g * G)) & 1) != 0;
  }
  return m;
}

// ---------------------------------------------------------------------------
// One workgroup: per sample, the key extent attended by covered rows and the
// KV heads involved; then items (sample, 128-key block, KV head) ordered by
// the number of attending rows, longest first, one queue per XCD keyed by
// (KV head, key block) so that an XCD streams the query blocks of few heads.
struct BwdPrep {
  const int64_t *cu;
  int64_t n;
  const libra_tile_t *tiles;
  int64_t T;
  int h_q, h_kv;
  int64_t n_q, n_kv;
  int32_t *hdr;
  int32_t *ext;
  unsigned long long *gmask;
  BwdItem *items;
  int64_t max_items;
  int grid;
  BwdSplit *splits;
  int32_t *cov, *cov_sum;   // per key block and KV head (see prep_bwd)
};
constexpr int kExtLds = 1024;   // samples whose extents and head sets are kept in LDS
constexpr int kMaxLong = 256;
constexpr int kPlaces = 2048;   // (key block, KV head) pairs whose covered rows are counted in LDS
struct BwdPrepLds {
  int32_t hist[kXcds * kQBuckets];
  int32_t part[kPrepThreads];
  int32_t cu[kCuLds];
  unsigned long long gmask[kExtLds];
  int32_t ext[kExtLds];
  int32_t longs[kMaxLong];
  int32_t cov_sum[kPlaces];
  uint16_t cuts[kPlaces], at[kExtLds];   // at: first place of a sample, in key blocks
  int32_t n_long, nslot, nsplit, tile_rows, taken, longest[2], block;
  unsigned long long covered, reached, work[2];
};
static_assert(kPlaces <= kXcds * kQBuckets, "the counts take the place of the histogram");
static_assert(sizeof(BwdPrepLds) <= 80 * 1024, "two preparation workgroups fit a CU");

__device__ __forceinline__ void prep_bwd(const BwdPrep &a, BwdPrepLds &lds) {
  const int64_t n = a.n, T = a.T, n_q = a.n_q, n_kv = a.n_kv;
  const int h_q = a.h_q, h_kv = a.h_kv;
  int32_t *hdr = a.hdr;
  const int tid = threadIdx.x;
  const int G = h_q / h_kv;
  const int R = h_kv >= kXcds ? 1 : kXcds / h_kv;
  const CuView cu = cu_view(a.cu, n, lds.cu);
  // extents and head sets gather in LDS when they fit, else in the workspace
  const bool in_lds = n <= kExtLds;
  int32_t *ext = in_lds ? lds.ext : a.ext;
  unsigned long long *gmask = in_lds ? lds.gmask : a.gmask;
  auto fence = [&]() {
    if (!in_lds) __threadfence();
    __syncthreads();
  };
  auto ext_of = [&](int64_t j) { return in_lds ? lds.ext[j] : ld_agent(&a.ext[j]); };
  // Atomics of all lanes on one counter in LDS: at an address that the compiler takes
  // for a lane's own.  Where it sees that there is one, it makes them a loop over
  // the lanes, about 1 us.
  auto at0 = [&](auto *p) {
    int z = 0;
    asm volatile("" : "+v"(z));
    return p + z;
  };
  auto gmask_of = [&](int64_t j) { return in_lds ? lds.gmask[j] : ld_agent(&a.gmask[j]); };
  for (int64_t j = tid; j < n; j += kPrepThreads) {
    __hip_atomic_store(&ext[j], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&gmask[j], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (tid == 0) {
    lds.n_long = lds.nslot = lds.nsplit = lds.tile_rows = lds.taken = 0;
    lds.covered = lds.reached = lds.work[0] = lds.work[1] = 0;
    lds.longest[0] = lds.longest[1] = lds.block = 0;
  }
  if (tid < 6) {
    // the skipped-tile count (counted here for the backward), the odd-heads
    // flag and the max |x| slots
    __hip_atomic_store(&hdr[tid == 0 ? (int)kBadTiles : tid == 1 ? (int)kOddHeads : kMaxAbs + tid - 2],
                       0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __threadfence();
  __syncthreads();
  int bad = 0, tile_rows = 0;
  bool odd = false;
  unsigned long long covered = 0;   // (row, head) pairs
  for (int64_t t = tid; t < T; t += kPrepThreads) {
    const libra_tile_t tl = a.tiles[t];
    if (!tile_ok(tl, n_q, n_kv, h_q)) {
      ++bad;
      continue;
    }
    tile_rows = max(tile_rows, (int)(tl.q_end - tl.q_begin));
    const unsigned long long bits = group_bits(tl.head_begin, tl.head_end, G, odd);
    for (int64_t j = upper_bound64(cu, n, tl.q_begin) - 1; j < n && cu[j] < tl.q_end; ++j) {
      const int64_t pe = tl.q_end < cu[j + 1] ? tl.q_end : cu[j + 1];
      const int64_t pb = tl.q_begin > cu[j] ? tl.q_begin : cu[j];
      atomicMax(&ext[j], (int32_t)(pe - cu[j]));
      atomicOr(&gmask[j], bits);
      if (pb < pe)
        covered += (unsigned long long)(unsigned)(pe - pb) *
                   (unsigned)(tl.head_end - tl.head_begin);
    }
  }
  if (covered) {
    atomicAdd(at0(&lds.covered), covered);
    atomicMax(at0(&lds.tile_rows), tile_rows);
  }
  if (bad) atomicAdd(&hdr[kBadTiles], bad);
  if (odd) atomicOr(&hdr[kOddHeads], 1);
  fence();
  // Samples of more than kCoopItems items are enumerated by the whole
  // workgroup (if the list of them overflows, each by a wave).  The others go to
  // the waves in groups of up to 64 that one load looks up, a sample to a lane;
  // a sample of no more items than its group has samples is enumerated by its
  // lane, the rest of the group one after another by the wave.  Every
  // enumeration sees the same items.  (One thread per sample took 82 us on a
  // 32K pack, whose 2,100 items lie in 9 samples; one wave per sample, each with
  // a lookup of its own, 8.0 ms on 65536 samples of one key block and 2 KV heads,
  // where groups take less than the dQ list beside them, 0.76.)
  constexpr int kCoopItems = 1024;
  const int group = (int)max((int64_t)1, min((int64_t)64, n / (kPrepThreads / 64)));
  auto blocks_of = [&](int32_t e) { return (e + kBwdBK - 1) / kBwdBK; };
  unsigned long long reached = 0;   // (row, head) pairs up to the extents
  for (int64_t j = tid; j < n; j += kPrepThreads) {
    const int32_t e = ext_of(j);
    if (in_lds) {
      a.ext[j] = e;   // for the passes over K and V
      lds.at[j] = (uint16_t)atomicAdd(at0(&lds.taken), blocks_of(e));
    }
    if (e) reached += (unsigned long long)e * (unsigned)(G * __builtin_popcountll(gmask_of(j)));
    if ((int64_t)blocks_of(e) * h_kv > kCoopItems) {
      const int32_t slot = atomicAdd(&lds.n_long, 1);
      if (slot < kMaxLong) lds.longs[slot] = (int32_t)j;
    }
  }
  if (reached) atomicAdd(at0(&lds.reached), reached);
  for (int i = tid; i < kPlaces; i += kPrepThreads) lds.hist[i] = 0;
  __syncthreads();
  const bool coop = lds.n_long <= kMaxLong;
  // item i of sample j: key block i / h_kv of KV head i % h_kv
  auto emit = [&](auto &&f, int64_t j, int32_t e, unsigned long long mk, int i) {
    const int kb = i / h_kv, g = i - kb * h_kv;
    if (mk >> g & 1ull)
      f(BwdItem{(int32_t)j, kb, g, -1, 0, INT32_MAX, 0, 0}, e, (g * R + kb % R) % kXcds);
  };
  // every whole item once: f(item, extent of its sample, queue)
  auto whole = [&](auto &&f) {
    const int l = tid & 63;
    int64_t j0 = (int64_t)(tid >> 6) * group, first = 0;   // next group; the current one
    int32_t e = 0;
    unsigned long long mk = 0, wide = 0;   // wide: samples of the group that the wave enumerates
    for (int k = 0;;) {
      int64_t j;
      int32_t ej;
      unsigned long long mj;
      int i, step;
      if (wide) {
        const int s = __builtin_ctzll(wide);
        wide &= wide - 1;
        j = first + s;
        ej = __shfl(e, s);
        mj = __shfl(mk, s);
        i = l;
        step = 64;
      } else if (j0 < n) {
        first = j0;
        j0 += kPrepThreads / 64 * group;
        j = first + l;
        const bool in = l < group && j < n;
        e = in ? ext_of(j) : 0;
        mk = in ? gmask_of(j) : 0;
        const int count = blocks_of(e) * h_kv;
        wide = __builtin_amdgcn_ballot_w64(count > group && !(coop && count > kCoopItems));
        ej = count <= group ? e : 0;
        mj = mk;
        i = 0;
        step = 1;
      } else if (coop && k < lds.n_long) {
        j = lds.longs[k++];
        ej = ext_of(j);
        mj = gmask_of(j);
        i = tid;
        step = kPrepThreads;
      } else {
        break;
      }
      for (const int count = blocks_of(ej) * h_kv; i < count; i += step) emit(f, j, ej, mj, i);
    }
  };
  // Split rows: when the longest item takes a quarter longer than the whole
  // call would if its work were spread evenly (few KV heads and samples: a 4K
  // pack has 70 items for 256 workgroups), the items longer than half of a
  // workgroup's share are cut into parts of C row blocks, summed by
  // bwd_dkdv_combine_kernel.  C is at least kBwdSplitMinBlocks and so large that
  // the parts fit the slots: items longer than C number at most work / C, their
  // parts twice that.  Below that line a part's own cost (K / V
  // loads, the fill of the ring, fp32 sums written and read) takes the gain:
  // 46 row blocks against a share of 4.6 (4K tokens, 2 KV heads, d = 64): 119 us
  // whole, 51 split; 430 against 391 (20K tokens, 4 KV heads): 908 and 935.
  //
  // Where the tiles cover every row of the samples up to their extents, an item is
  // as long as the extent past its first key.  Elsewhere (a context-parallel share,
  // a single tile, a pool worker's tiles) the extent is only a bound: when the line is
  // crossed by the extents, the steps of the covered rows are counted, and rule and
  // cuts go by them, so that no part is without rows.  (By extents, 446 of the 553
  // parts of a 3K-row share of 48K tokens with 4 / 1 heads were: its backward took
  // 267 us, now 180; a tile of 2400 rows deep in a 48K sample 245, now 206, uncut.)
  auto by_extent = [&](const BwdItem &it, int32_t e) {
    return (e - it.kb * kBwdBK + kRows - 1) / kRows;
  };
  // longest item and sum of all (pass 0: by extent, 1: by steps): crosses the line?
  auto crosses = [&](int pass, auto &&cost) {
    unsigned long long w = 0;
    int32_t m = 0;
    whole([&](const BwdItem &it, int32_t e, int) {
      const int c = cost(it, e);
      w += (unsigned long long)c;
      m = max(m, c);
    });
    if (m) {
      atomicAdd(at0(&lds.work[pass]), w);
      atomicMax(at0(&lds.longest[pass]), m);
    }
    __syncthreads();
    return 4ull * (unsigned)lds.longest[pass] * (unsigned)a.grid > 5ull * lds.work[pass] &&
           lds.longest[pass] >= 2 * kBwdSplitMinBlocks;
  };
  // Steps (32 covered rows x two heads of one tile), times 32, of each (sample, key
  // block, KV head): `cov` those of the block's own 128 rows, cov_sum those of all
  // rows from it on, which attend it; in LDS if the key blocks reached fit there, else
  // in the workspace, where a sample's places come past those of the samples before it.
  const bool cov_lds = in_lds && (int64_t)lds.taken * h_kv <= kPlaces;
  auto lds_place = [&](int j, int kb, int g) { return (lds.at[j] + kb) * h_kv + g; };
  auto ws_place = [&](int64_t j, int kb, int g) { return (cu[j] / kBwdBK + j + kb) * h_kv + g; };
  auto steps_of = [&](int j, int kb, int g) {
    return (unsigned)(cov_lds ? lds.cov_sum[lds_place(j, kb, g)]
                              : ld_agent(&a.cov_sum[ws_place(j, kb, g)]));
  };
  auto sync_cov = [&]() {
    if (!cov_lds) __threadfence();
    __syncthreads();
  };
  bool split = crosses(0, by_extent), counted = split && lds.covered != lds.reached;
  if (counted) {
    if (!cov_lds) {
      whole([&](const BwdItem &it, int32_t, int) { a.cov[ws_place(it.sample, it.kb, it.g)] = 0; });
      sync_cov();
    }
    const int64_t windows = (lds.tile_rows + kBwdBK - 1) / kBwdBK;
    for (int64_t v = tid; v < T * windows; v += kPrepThreads) {
      const bool small = T * windows < INT32_MAX;   // a 32-bit division, not a 64-bit one
      const int64_t t = small ? (int64_t)((uint32_t)v / (uint32_t)windows) : v / windows;
      const libra_tile_t tl = a.tiles[t];
      if (!tile_ok(tl, n_q, n_kv, h_q)) continue;
      const int64_t wa = tl.q_begin + kBwdBK * (v - t * windows);
      const int64_t wb = wa + kBwdBK < tl.q_end ? wa + kBwdBK : tl.q_end;
      if (wa >= wb) continue;
      for (int64_t j = upper_bound64(cu, n, wa) - 1; j < n && cu[j] < wb; ++j) {
        const int la = (int)((wa > cu[j] ? wa : cu[j]) - cu[j]);
        const int lb = (int)((wb < cu[j + 1] ? wb : cu[j + 1]) - cu[j]);
        for (int kb = la / kBwdBK; kb * kBwdBK < lb && la < lb; ++kb) {
          const int rows = min(lb, kb * kBwdBK + kBwdBK) - max(la, kb * kBwdBK);
          for (int g = tl.head_begin / G; g * G < tl.head_end; ++g) {
            const int nh = min(tl.head_end, (g + 1) * G) - max(tl.head_begin, g * G);
            const int x = rows * ((nh + 1) / 2);
            if (cov_lds) atomicAdd(&lds.hist[lds_place((int)j, kb, g)], x);
            else atomicAdd(&a.cov[ws_place(j, kb, g)], x);
          }
        }
      }
    }
    sync_cov();
    // The sums block by block (the line is crossed by samples of at most some 400
    // blocks), kept below 2^31 whatever overlapping tiles count; and the most that
    // one block holds
    int most_block = 0;
    split = crosses(1, [&](const BwdItem &it, int32_t e) {
      const int count = blocks_of(e) - it.kb;
      const unsigned most = 0x7fffffffu / (unsigned)blocks_of(e);
      unsigned s = 0;
      auto add = [&](int x) { s += min((unsigned)x, most); };
      if (cov_lds) {
        const int at = lds_place(it.sample, it.kb, it.g);
#pragma unroll 16
        for (int i = 0; i < count; ++i) add(lds.hist[at + i * h_kv]);
        most_block = max(most_block, lds.hist[at]);
        lds.cov_sum[at] = (int32_t)s;
      } else {
        const int64_t at = ws_place(it.sample, it.kb, it.g);
#pragma unroll 8
        for (int i = 0; i < count; ++i) add(ld_agent(&a.cov[at + (int64_t)i * h_kv]));
        most_block = max(most_block, ld_agent(&a.cov[at]));
        a.cov_sum[at] = (int32_t)s;
      }
      return (int)((s + kRows - 1) / kRows);
    });
    if (most_block) atomicMax(at0(&lds.block), most_block);
    counted = split;   // else every item stays whole, ordered by extent
    sync_cov();
  }
  // C; 0: no item is split.  By extent, it is half of a workgroup's share, and the
  // parts of an item are equal row ranges.  By steps, items are cut from the last
  // row back, so that those of a sample share their cuts: C each, and the first
  // one takes the rest.  Such parts fill the workgroups better when they are a
  // little more than a whole share, so that there are no more of them than
  // workgroups: counted on the host, 82 calls take 0.78 of the time of cuts by extent,
  // 0.82 with a share exactly, 0.82 with 1.25 and 0.84 with half a share.  C is no less
  // than one key block's steps, so that a part has rows.
  const unsigned long long work = lds.work[counted];
  const unsigned block = (unsigned)lds.block;
  const int least = max(kBwdSplitMinBlocks, counted ? (int)((block + kRows - 1) / kRows) : 0);
  const int chunk =
      split ? (int)max(counted ? (work + work / 16) / (unsigned)a.grid
                               : work / (2ull * (unsigned)a.grid),
                       max((2 * work + kBwdSplitSlots - 1) / kBwdSplitSlots,
                           (unsigned long long)least))
            : 0;
  const unsigned part = (unsigned)min((unsigned long long)chunk * kRows, 1ull << 31);
  // Cut m of a (sample, KV head), in blocks of 32 rows: the first key block from which
  // on there are no more than m C steps, or inside the one before it if that is as
  // full as any, so that m C remain.  It takes the place of key block m, where the
  // counts are not needed any more.  Written in the counting pass of build_queues, by
  // the items before and after which it lies, for every m that an item can ask for.
  auto write_cuts = [&](const BwdItem &it, int nb, unsigned s0) {
    const int next = it.kb + 1;
    const unsigned s1 = next < nb ? steps_of(it.sample, next, it.g) : 0;
    for (unsigned m = max(1u, (s1 + part - 1) / part); m < (unsigned)nb && m * part < s0; ++m) {
      const unsigned more = s0 - s1 == block ? (m * part - s1) * 4ull / block : 0;   // < 4
      const int c = kBwdBK / kRows * next - (int)more;
      if (cov_lds) lds.cuts[lds_place(it.sample, (int)m, it.g)] = (uint16_t)c;
      else a.cov[ws_place(it.sample, (int)m, it.g)] = c;
    }
    if (!cov_lds) __threadfence();
  };
  auto cut = [&](int j, int g, int m) {
    return kRows * (cov_lds ? lds.cuts[lds_place(j, m, g)] : ld_agent(&a.cov[ws_place(j, m, g)]));
  };
  auto each = [&](auto &&f, bool scatter) {
    whole([&](const BwdItem &it, int32_t e, int x) {
      int cost = by_extent(it, e), np = 1, per = chunk;
      if (counted) {
        const unsigned s = steps_of(it.sample, it.kb, it.g);
        cost = (int)((s + kRows - 1) / kRows);
        np = max(1, min((int)((s + part - 1) / part), blocks_of(e) - it.kb));
        if (!scatter) write_cuts(it, blocks_of(e), s);
      } else if (chunk && cost > chunk) {
        np = (cost + chunk - 1) / chunk;
        per = (cost + np - 1) / np;
      }
      int32_t base = 0;
      if (scatter && np > 1) {
        base = atomicAdd(at0(&lds.nslot), np);
        a.splits[atomicAdd(&lds.nsplit, 1)] = BwdSplit{it, base, np, 0, 0};
      }
      // the odd part: the first one by steps, the last one by extent
      const int odd_part = counted ? 0 : np - 1, odd_cost = max(cost - per * (np - 1), 1);
      BwdItem ip = it;
      for (int p = 0; p < np; ++p) {
        if (scatter && np > 1) {
          ip.slot = base + p;
          ip.r0 = p ? ip.r1 : it.kb * kBwdBK;
          ip.r1 = p + 1 == np ? INT32_MAX
                  : counted   ? cut(it.sample, it.g, np - 1 - p)
                              : ip.r0 + kRows * per;
        }
        f(ip, (int64_t)(p == odd_part ? odd_cost : per), x);
      }
    });
  };
  build_queues<BwdItem>(each, lds.hist, lds.part, hdr, kBwdQ, kBadTiles, a.items, a.max_items,
                        a.grid);
  __syncthreads();
  if (tid == 0) hdr[kBwdSplits] = lds.nsplit;
}

// Both preparation passes of a call, side by side: workgroup 0 builds the
// dK / dV items, workgroup 1 the dQ items.
__global__ __launch_bounds__(kPrepThreads) void prep_bwd_kernel(BwdPrep b, FwdPrep f) {
  __shared__ union Lds {
    BwdPrepLds b;
    FwdPrepLds f;
  } lds;
  if (blockIdx.x == 0) prep_bwd(b, lds.b);
  else prep_fwd(f, lds.f);
}

// ---------------------------------------------------------------------------
// fp16 operands of the dK / dV kernel.  Its products run on fp16 copies of
// Q, dO, K and V (same matrix-core rate as bf16, three more significant bits
// for the rounded P and dS operands), each scaled by a power of two chosen
// from the tensor's max |x| over what the kernel reads (fp16_scale), so that
// the copies stay inside the fp16 range whatever the inputs' magnitude.
// Two passes find the maxima (fp32 bits, atomicMax on the header slots
// kMaxAbs + 0..3): Q and dO over the covered (row, head) pairs, K and V over
// the keys of the dK / dV work items.

// Workgroup-wide max of two non-negative floats (256 threads), then at most
// one atomic per slot and workgroup, skipped when the slot already holds as
// much (fp32 bits of non-negative floats order like unsigned integers).  Per
// wave atomics on the same two slots serialise: thousands of them took
// longer than the pass's loads.
__device__ __forceinline__ void block_max2_to(float a, float b, int32_t *slot_a,
                                              int32_t *slot_b) {
  __shared__ float red[2][4];
  for (int o = 32; o > 0; o >>= 1) {
    a = fmaxf(a, __shfl_xor(a, o));
    b = fmaxf(b, __shfl_xor(b, o));
  }
  const int tid = threadIdx.x;
  if ((tid & 63) == 0) {
    red[0][tid >> 6] = a;
    red[1][tid >> 6] = b;
  }
  __syncthreads();
  if (tid == 0) {
    a = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    b = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    const unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
    if (a > 0.f && ua > (unsigned)ld_agent(slot_a))
      atomicMax(reinterpret_cast<unsigned int *>(slot_a), ua);
    if (b > 0.f && ub > (unsigned)ld_agent(slot_b))
      atomicMax(reinterpret_cast<unsigned int *>(slot_b), ub);
  }
}

__device__ __forceinline__ float absmax8(const bf16x8 &x) {
  float m = 0.f;
  static_for<8>([&](auto i) { m = fmaxf(m, fabsf(static_cast<float>(x[int(i)]))); });
  return m;
}

constexpr int kTileSplit = 64;

// Per tile (kTileSplit workgroups each): max |Q| and max |dO| over the
// covered (row, head) pairs; and, in the records, zeros for the rows of the
// tile's first and last 32-row blocks that lie outside the tile (the dK / dV
// kernel stages whole records; rows no tile covers must hold finite values,
// since they meet P = dS = 0 in its products).  So must the -D operand of a tile's
// rows past the last sample (position `pool` on), which no dQ item writes.
template <int D>
__device__ __forceinline__ void absmax_q(unsigned block, const bf16 *__restrict__ q,
                                         const bf16 *__restrict__ dout,
                                         const libra_tile_t *__restrict__ tiles, int h_q,
                                         int64_t n_q, int64_t n_kv, int64_t pool,
                                         int32_t *__restrict__ hdr, f16 *__restrict__ rec) {
  const int tid = threadIdx.x;
  const libra_tile_t tl = tiles[block / kTileSplit];
  if (!tile_ok(tl, n_q, n_kv, h_q)) return;
  const int64_t ra = tl.q_row, rb = tl.q_row + (tl.q_end - tl.q_begin);
  const int r = tid >> 3, part = tid & 7;   // 8 threads per row, 32 rows per pass
  const int64_t past = tl.q_row + (pool - tl.q_begin);   // first row past the last sample
  float mq = 0.f, mo = 0.f;
  for (int64_t m = ra / kRows + block % kTileSplit; m * kRows < rb; m += kTileSplit) {
    const int64_t row = m * kRows + r;
    const bool ok = row >= ra && row < rb;
    for (int h = tl.head_begin; h < tl.head_end; ++h) {
      f16 *rp = rec + ((size_t)m * h_q + h) * rec_els(D);
      f16x8 z;
      static_for<8>([&](auto i) { z[int(i)] = f16(0.f); });
      f16 *ag = rp + 2 * kRows * D + 8 * perm32(r);   // the row's lanes of both operands
      if (ok) {
        if (row >= past && part == 0) *reinterpret_cast<f16x8 *>(ag + 2 * (kAugEl / 4)) = z;
        const size_t off = ((size_t)row * h_q + h) * D + part * (D / 8);
        static_for<D / 64>([&](auto c) {
          mq = fmaxf(mq, absmax8(*reinterpret_cast<const bf16x8 *>(q + off + 8 * c)));
          mo = fmaxf(mo, absmax8(*reinterpret_cast<const bf16x8 *>(dout + off + 8 * c)));
        });
        continue;
      }
      static_for<D / 64>([&](auto c) {
        const int at = rec_at(r, part * (D / 64) + c);
        *reinterpret_cast<f16x8 *>(rp + at) = z;
        *reinterpret_cast<f16x8 *>(rp + kRows * D + at) = z;
      });
      if (part < 4) *reinterpret_cast<f16x8 *>(ag + part * (kAugEl / 4)) = z;
    }
  }
  block_max2_to(mq, mo, &hdr[kMaxAbs + 0], &hdr[kMaxAbs + 1]);
}

// The keys the dK / dV kernel loads: for every sample with covered rows,
// its keys up to the end of the last 128-key block that those rows attend
// (all KV heads).  One wave per key row.  CONVERT = false: max |K| and
// max |V| over them; CONVERT = true: their scaled fp16 copies.
template <int D, bool CONVERT>
__device__ __forceinline__ void kv_pass(unsigned block, unsigned blocks,
                                        const bf16 *__restrict__ k, const bf16 *__restrict__ v,
                                        const int64_t *__restrict__ cu, int64_t n,
                                        const int32_t *__restrict__ ext, int h_kv, int64_t n_kv,
                                        int32_t *__restrict__ hdr, f16 *__restrict__ k16,
                                        f16 *__restrict__ v16) {
  const int l = threadIdx.x & 63;
  const int64_t wave = ((int64_t)block * 256 + threadIdx.x) >> 6;
  const int64_t waves = (int64_t)blocks * 4;
  const int chunks = h_kv * D / 8;   // 16-byte chunks of a row
  float mk = 0.f, mv = 0.f, s_k = 1.f, s_v = 1.f;
  if constexpr (CONVERT) {
    s_k = fp16_scale((uint32_t)hdr[kMaxAbs + 2], false);
    s_v = fp16_scale((uint32_t)hdr[kMaxAbs + 3], true);
  }
  int64_t lo = 0, hi = 0, end = 0;   // rows [lo, hi) of the current sample; loaded keys end at `end`
  for (int64_t row = wave; row < n_kv; row += waves) {
    if (row < lo || row >= hi) {
      const int64_t j = upper_bound64(cu, n, row) - 1;
      lo = cu[j];
      hi = cu[j + 1];
      const int64_t e = (int64_t)ext[j];
      const int64_t lim = (e + kBwdBK - 1) / kBwdBK * kBwdBK;
      end = lo + (e > 0 ? (lim < hi - lo ? lim : hi - lo) : 0);
    }
    if (row >= end) continue;
    for (int c = l; c < chunks; c += 64) {
      const size_t off = (size_t)row * h_kv * D + 8 * (size_t)c;
      const bf16x8 kx = *reinterpret_cast<const bf16x8 *>(k + off);
      const bf16x8 vx = *reinterpret_cast<const bf16x8 *>(v + off);
      if constexpr (CONVERT) {
        f16x8 kh, vh;
        static_for<8>([&](auto i) {
          kh[int(i)] = static_cast<f16>(static_cast<float>(kx[int(i)]) * s_k);
          vh[int(i)] = static_cast<f16>(static_cast<float>(vx[int(i)]) * s_v);
        });
        *reinterpret_cast<f16x8 *>(k16 + off) = kh;
        *reinterpret_cast<f16x8 *>(v16 + off) = vh;
      } else {
        mk = fmaxf(mk, absmax8(kx));
        mv = fmaxf(mv, absmax8(vx));
      }
    }
  }
  if constexpr (!CONVERT) {
    block_max2_to(mk, mv, &hdr[kMaxAbs + 2], &hdr[kMaxAbs + 3]);
  }
}

// Pre-pass over the covered (row, head) pairs, 32 rows at a time:
//   * the records of the dK / dV kernel: the fp16 copies of Q and dO (scaled,
//     see above) and the first of the two operands of its extra 16-deep
//     k-block: MFMA A-operand lane l < 32 holds three fp16 terms summing to
//     -LSE / scale (first operand) or -D (second, written by the dQ kernel
//     from the exact row sums) of the block's row perm32(l), in the scaled
//     units of the copies, then zeros; lanes 32..63 hold zeros.  Against a B
//     operand of ones in k = 0, 1, 2 the products then come out as
//     S - LSE / scale and dP - D directly;
//   * the 32 values LSE * log2(e) followed by the 32 values D = rowsum(dO * O)
//     of each block and head for the dQ kernel ("stats",
//     [h_q][nq_pad / 32][64] floats, so one 256-byte load fetches both).
template <int D>
__device__ __forceinline__ void pre_pass(unsigned block, const bf16 *__restrict__ q,
                                         const bf16 *__restrict__ o,
                                         const bf16 *__restrict__ dout,
                                         const float *__restrict__ lse,
                                         const libra_tile_t *__restrict__ tiles, int h_q,
                                         int64_t n_q, int64_t n_kv, int64_t nq_pad, float scale,
                                         const int32_t *__restrict__ hdr,
                                         f16 *__restrict__ rec, float *__restrict__ stats) {
  const int tid = threadIdx.x;
  const libra_tile_t tl = tiles[block / kTileSplit];
  if (!tile_ok(tl, n_q, n_kv, h_q)) return;
  const float s_q = fp16_scale((uint32_t)hdr[kMaxAbs + 0], false);
  const float s_o = fp16_scale((uint32_t)hdr[kMaxAbs + 1], true);
  const float s_k = fp16_scale((uint32_t)hdr[kMaxAbs + 2], false);
  const int64_t ra = tl.q_row, rb = tl.q_row + (tl.q_end - tl.q_begin);
  // 8 threads per row, 32 rows per pass
  const int r = tid >> 3, part = tid & 7;
  for (int64_t m = ra / kRows + block % kTileSplit; m * kRows < rb; m += kTileSplit) {
    const int64_t row = m * kRows + r;
    const bool ok = row >= ra && row < rb;
    for (int h = tl.head_begin; h < tl.head_end; ++h) {
      float acc = 0.f;
      f16 *rp = rec + ((size_t)m * h_q + h) * rec_els(D);
      if (ok) {
        const size_t off = ((size_t)row * h_q + h) * D + part * (D / 8);
        static_for<D / 64>([&](auto c) {
          const bf16x8 qv = *reinterpret_cast<const bf16x8 *>(q + off + 8 * c);
          const bf16x8 ov = *reinterpret_cast<const bf16x8 *>(o + off + 8 * c);
          const bf16x8 dv = *reinterpret_cast<const bf16x8 *>(dout + off + 8 * c);
          f16x8 qh, dh;
          static_for<8>([&](auto i) {
            const float dx = static_cast<float>(dv[int(i)]);
            acc += static_cast<float>(ov[int(i)]) * dx;
            qh[int(i)] = static_cast<f16>(static_cast<float>(qv[int(i)]) * s_q);
            dh[int(i)] = static_cast<f16>(dx * s_o);
          });
          const int at = rec_at(r, part * (D / 64) + c);
          *reinterpret_cast<f16x8 *>(rp + at) = qh;
          *reinterpret_cast<f16x8 *>(rp + kRows * D + at) = dh;
        });
      }
      acc += __shfl_xor(acc, 1);
      acc += __shfl_xor(acc, 2);
      acc += __shfl_xor(acc, 4);
      if (part == 0 && ok) {
        float *st = stats + ((size_t)h * (nq_pad / kRows) + m) * 2 * kRows;
        const float lv = lse[(size_t)h * n_q + row];
        st[r] = lv * kLog2e;
        st[kRows + r] = acc;
        f16x8 sv;
        split3h(-lv / scale * (s_q * s_k), sv);
        f16 *ag = rp + 2 * kRows * D + 8 * perm32(r);
        *reinterpret_cast<f16x8 *>(ag) = sv;
        static_for<8>([&](auto i) { sv[int(i)] = f16(0.f); });
        *reinterpret_cast<f16x8 *>(ag + kAugEl / 4) = sv;
        *reinterpret_cast<f16x8 *>(ag + 3 * (kAugEl / 4)) = sv;
      }
    }
  }
}

__device__ __forceinline__ void zero_fill(unsigned block, unsigned blocks, uint4 *__restrict__ p,
                                          int64_t n16) {
  for (int64_t i = (int64_t)block * 256 + threadIdx.x; i < n16; i += (int64_t)blocks * 256)
    p[i] = make_uint4(0, 0, 0, 0);
}
__global__ __launch_bounds__(256) void zero_kernel(uint4 *__restrict__ p, int64_t n16) {
  zero_fill(blockIdx.x, gridDim.x, p, n16);
}

// The passes before the dQ and dK / dV kernels, in two launches: what needs
// nothing but the extents (max |x| of Q, dO, K and V; zero dK and dV in bf16
// mode), then what needs the maxima (the fp16 copies and records).  Each part
// takes its own range of workgroups.  In launches of their own, the parts of a
// 4K pack's backward took 4 to 24 us each for work of 1 to 3 us.
struct BwdPass {
  const bf16 *q, *k, *v, *o, *dout;
  const float *lse;
  const int64_t *cu;
  int64_t n;
  const libra_tile_t *tiles;
  int h_q, h_kv;
  int64_t n_q, n_kv, nq_pad;
  float scale;
  int32_t *hdr;
  const int32_t *ext;
  f16 *rec, *k16, *v16;
  float *stats;
  uint4 *dk, *dv;                          // to be zeroed
  int64_t n16;                             // 16-byte pieces of each
  unsigned tile_blocks, kv_blocks, zero_blocks;
};
template <int D>
__global__ __launch_bounds__(256) void bwd_max_kernel(BwdPass a) {
  unsigned b = blockIdx.x;
  if (b == 0 && threadIdx.x == 0 && a.hdr[kDqFull]) atomicAdd(&a.hdr[kBadTiles], 1);
  if (b < a.kv_blocks) {
    kv_pass<D, false>(b, a.kv_blocks, a.k, a.v, a.cu, a.n, a.ext, a.h_kv, a.n_kv, a.hdr, a.k16,
                      a.v16);
  } else if ((b -= a.kv_blocks) < a.tile_blocks) {
    absmax_q<D>(b, a.q, a.dout, a.tiles, a.h_q, a.n_q, a.n_kv, a.cu[a.n], a.hdr, a.rec);
  } else {
    b -= a.tile_blocks;
    const unsigned half = a.zero_blocks / 2;
    zero_fill(b % half, half, b < half ? a.dk : a.dv, a.n16);
  }
}
template <int D>
__global__ __launch_bounds__(256) void bwd_copy_kernel(BwdPass a) {
  const unsigned b = blockIdx.x;
  if (b < a.kv_blocks)
    kv_pass<D, true>(b, a.kv_blocks, a.k, a.v, a.cu, a.n, a.ext, a.h_kv, a.n_kv, a.hdr, a.k16,
                     a.v16);
  else
    pre_pass<D>(b - a.kv_blocks, a.q, a.o, a.dout, a.lse, a.tiles, a.h_q, a.n_q, a.n_kv, a.nq_pad,
                a.scale, a.hdr, a.rec, a.stats);
}

// ---------------------------------------------------------------------------
// dK / dV kernel.
template <int D>
struct KvShape {
  static constexpr int Q_EL = kRows * D;
  static constexpr int HEAD_EL = rec_els(D);                  // Q, dO, aug of one head
  static constexpr int STAGE_EL = 2 * HEAD_EL;                // a step is two query heads
  static constexpr int NSTAGE = 4;                            // LDS ring of steps
  static_assert((NSTAGE & (NSTAGE - 1)) == 0, "ring index by mask");
  static constexpr int LOADS = STAGE_EL / 512 / kWaves;       // 1 KiB copies per wave per step
  static_assert(LOADS * 512 * kWaves == STAGE_EL, "every wave copies as much");
  static constexpr size_t SMEM = NSTAGE * STAGE_EL * sizeof(bf16);
  static_assert((NSTAGE - 2) * LOADS <= 63, "vmcnt range");
};

// Walks the steps (32-row query block x two query heads) that attend one KV
// block: tiles in list order, query blocks in row order, heads in order.  Per
// fragment (one tile's rows of the sample) everything a step needs is
// precomputed, so that advancing is a few 32-bit scalar operations plus one
// running 64-bit record offset.
struct StepIter {
  const libra_tile_t *tiles;
  int64_t T, n_q, n_kv, key0, p0, p1;   // rows at positions [p0, p1)
  int h_q, g, G, kloc0, rkib;   // rkib: KiB of a record
  // fragment
  int64_t t;                // tile index
  int nm, lo0, hin, qb0;    // blocks; lo of block 0; hi of the last block; q_loc of its row 0
  int h0, h1;
  // position
  int mi, h;
  int64_t rec;              // offset of the record of (block, h), in KiB
  bool valid;

  __device__ bool seek() {
    for (; t < T; ++t) {
      const libra_tile_t tl = tiles[t];
      if (!tile_ok(tl, n_q, n_kv, h_q)) continue;
      const int64_t pb = tl.q_begin > p0 ? tl.q_begin : p0;
      const int64_t pe = tl.q_end < p1 ? tl.q_end : p1;
      if (pb >= pe) continue;
      h0 = max(tl.head_begin, g * G);
      h1 = min(tl.head_end, (g + 1) * G);
      if (h0 >= h1) continue;
      const int64_t fra = tl.q_row + (pb - tl.q_begin);
      const int64_t frb = fra + (pe - pb);
      const int64_t qla = pb - key0;
      const int64_t first = fra + (kloc0 > qla ? kloc0 - qla : 0);
      if (first >= frb) continue;
      const int64_t mf = first / kRows, ml = (frb - 1) / kRows;
      const int64_t row0 = mf * kRows;
      nm = (int)(ml - mf + 1);
      lo0 = (int)(fra > row0 ? fra - row0 : 0);
      hin = (int)(frb - ml * kRows);
      qb0 = (int)(qla - (fra - row0));
      mi = 0;
      h = h0;
      rec = (mf * h_q + h0) * rkib;
      return true;
    }
    return false;
  }
  __device__ void start() { t = 0; valid = seek(); }
  // steps are pairs of query heads (h, h + 1); two() is false for the last
  // step of an odd head count
  __device__ void next() {
    if ((h += 2) < h1) {
      rec += 2 * rkib;
      return;
    }
    rec += (int64_t)((h_q - (h - 2 - h0)) * rkib);   // back by the heads advanced within this block
    h = h0;
    if (++mi < nm) return;
    ++t;
    valid = seek();
  }
  __device__ bool two() const { return h + 1 < h1; }
  __device__ int lo() const { return mi == 0 ? lo0 : 0; }
  __device__ int hi() const { return mi == nm - 1 ? hin : kRows; }
  __device__ int qb() const { return qb0 + kRows * mi; }        // q_loc of the block's row 0
};

template <int D>
__global__ __launch_bounds__(kThreads, 1) __attribute__((amdgpu_waves_per_eu(1, 1))) void attn_bwd_dkdv_kernel(
    const f16 *__restrict__ k, const f16 *__restrict__ v, const f16 *__restrict__ rec,
    const int64_t *__restrict__ cu, const libra_tile_t *__restrict__ tiles, int64_t T,
    const BwdItem *__restrict__ items, int32_t *__restrict__ hdr, int h_q, int h_kv,
    int64_t n_q, int64_t n_kv, float scale, float c2, void *__restrict__ dk_out,
    void *__restrict__ dv_out, int accumulate, float *__restrict__ parts) {
  using S = KvShape<D>;
  extern __shared__ __attribute__((aligned(16))) bf16 smem[];
  __shared__ int32_t s_item;

  const int tid = threadIdx.x, l = tid & 63, ln = l & 31, kg = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index (uniform)
  const int G = h_q / h_kv;
  const int q_serve = xcd_of_workgroup();
  int q_state = kTakeFirst;
  // per-lane LDS offsets (elements) of the operand reads: rows of Q / dO for
  // S and dP (row perm32(ln), chunk 2 c + kg; one offset per parity of c), and
  // the transpose reads that give dO^T / Q^T for dV^T and dK^T: this lane
  // addresses 4 columns of row 8 kg + 4 half + i of the block (i = (l % 16) /
  // 4), the columns whose 16-lane group hands them to the lanes that need
  // column perm32(ln) (one offset per half)
  const int prow = perm32(ln);
  const int qoff[2] = {rec_at(prow, kg), rec_at(prow, 2 + kg)};
  int troff[2];
  {
    const int grp = l >> 4, i = (l & 15) >> 2, r = l & 3;
    static_for<2>([&](auto hf) {
      troff[hf] = rec_at(8 * (grp >> 1) + 4 * hf + i, 2 * (grp & 1) + (r & 1)) + 4 * (r >> 1);
    });
  }
  // B operand of the augmented k-block: ones in k = 0, 1, 2 (lanes of kg 0)
  f16x8 ones3;
  static_for<8>([&](auto i) { ones3[int(i)] = f16(kg == 0 && i < 3 ? 1.f : 0.f); });
  // Every operand is an fp16 copy scaled by a power of two (fp16_scale): the
  // scores come out multiplied by s_q s_k, dP and D by s_o s_v, so the
  // exponent takes c2 / (s_q s_k) and the outputs are scaled back at the end
  // (exactly: all factors are powers of two).
  const bool odd_heads = hdr[kOddHeads] != 0;
  const float s_q = fp16_scale((uint32_t)hdr[kMaxAbs + 0], false);
  const float s_o = fp16_scale((uint32_t)hdr[kMaxAbs + 1], true);
  const float s_k = fp16_scale((uint32_t)hdr[kMaxAbs + 2], false);
  const float s_v = fp16_scale((uint32_t)hdr[kMaxAbs + 3], true);
  const float c2s = c2 / (s_q * s_k);
  const float dk_mul = scale / (s_q * s_o * s_v), dv_mul = 1.f / s_o;

  for (;;) {
    if (w == 0) {
      const int got = take_item(hdr, kBwdQ, q_serve, q_state);
      if (tid == 0) s_item = got;
    }
    __syncthreads();
    const int idx = __builtin_amdgcn_readfirstlane(s_item);
    if (idx < 0) break;
    const BwdItem item = items[idx];
    const int64_t key0 = cu[item.sample];
    const int64_t len = cu[item.sample + 1] - key0;
    const int g = item.g;
    const int kloc0 = item.kb * kBwdBK;
    const int kw0 = kloc0 + 32 * w;                   // first key of this wave
    const int kl = kw0 + ln;                          // this lane's key (sample-local)
    const bool key_ok = kl < len;
    const bool wave_keys_ok = kw0 + 31 < len;
    const int64_t krow = key0 + kl;

    f16x8 kf[D / 16], vf[D / 16];
    static_for<D / 16>([&](auto c) {
      if (key_ok) {
        const size_t off = ((size_t)krow * h_kv + g) * D + 16 * c + 8 * kg;
        kf[c] = *reinterpret_cast<const f16x8 *>(k + off);
        vf[c] = *reinterpret_cast<const f16x8 *>(v + off);
      } else {
        static_for<8>([&](auto i) { kf[c][int(i)] = f16(0.f); vf[c][int(i)] = f16(0.f); });
      }
    });
    wait_vm_known();
    f32x16 dva[D / 32], dka[D / 32];
    static_for<D / 32>([&](auto dt) {
      dva[dt] = mfma_zero();
      dka[dt] = mfma_zero();
    });

    // ---- one step = (32-row query block, two heads): the records of heads h
    // and h + 1, contiguous, go global -> LDS into ring stage `sg`, a quarter
    // by each wave (a step of one head copies the record after its own too:
    // not computed; rows of the block outside the fragment are rows of other
    // fragments or zeros, their P and dS are masked to zero)
    const char *cp_src = nullptr;   // the step being copied
    uint32_t cp_dst = 0;
    auto copy_part = [&](auto part) {
      constexpr int at = S::LOADS * part / 3, n = S::LOADS * (part + 1) / 3 - at;
      g2l_run<n>(cp_src + 1024 * at, 16u * l, cp_dst + 1024u * at);
    };
    auto copy_all = [&]() { static_for<3>([&](auto part) { copy_part(part); }); };

    // ---- compute one step from the LDS stage at Qs.  Rows of the block are
    // m0 + iq, iq in [0, 32); with MASK, row iq counts for this lane's key
    // only when lower <= iq < upper (inside the fragment and causal).
    auto step = [&](auto copy_t, bool full, const bf16 *Qs, int lower, int upper) {
      constexpr bool COPY = decltype(copy_t)::value;   // posts the copies of the iteration
      constexpr int NC = D / 16, NT = D / 32;
      const bf16 *Ag = Qs + 2 * S::Q_EL + 8 * l;   // -LSE / scale operand, then the -D operand
      // Q rows, then (at Q_EL) dO rows; the transpose reads of Q^T, then dO^T
      const bf16 *rp[2] = {Qs + qoff[0], Qs + qoff[1]};
      const f16 *tp[2] = {reinterpret_cast<const f16 *>(Qs) + troff[0],
                          reinterpret_cast<const f16 *>(Qs) + troff[1]};
      // (1) Q rows and this lane's part of the -LSE / scale operand
      f16x8 qa[NC], oa[NC], sag, dag;
      sag = *reinterpret_cast<const f16x8 *>(Ag);
      static_for<NC>([&](auto c) {
        qa[c] = *reinterpret_cast<const f16x8 *>(rp[c & 1] + 1024 * (c >> 1));
      });
      __builtin_amdgcn_sched_barrier(0);
      // (2) S - LSE / scale = [Q | aug] [K | ones]^T (queries on M, this
      // lane's key on N) while the dO rows and the -D operand load
      f32x16 sa = mfma32h(sag, ones3, mfma_zero_c()), pa;
      static_for<NC>([&](auto c) { sa = mfma32h(qa[c], kf[c], sa); });
      dag = *reinterpret_cast<const f16x8 *>(Ag + kAugEl / 2);
      static_for<NC>([&](auto c) {
        oa[c] = *reinterpret_cast<const f16x8 *>(rp[c & 1] + S::Q_EL + 1024 * (c >> 1));
      });
      static_for<NC + 1>([&](auto i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, i < NC / 2 + 1 ? 2 : 0, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (COPY) copy_part(std::integral_constant<int, 0>{});
      // (3) dP - D = [dO | aug] [V | ones]^T with P = exp2((S - LSE / scale) c2)
      // on the VALU and the transpose reads of dO^T; register 8 hh + i of S
      // holds row 16 hh + 8 kg + i
      f16x8 ta[NT][2];
      float pf[16];
      f16x8 pb16[2], db16[2];
      auto phase3 = [&](auto mask_t) {
      constexpr bool MASK = decltype(mask_t)::value;
      pa = mfma32h(dag, ones3, mfma_zero_c());
      static_for<NC>([&](auto c) { pa = mfma32h(oa[c], vf[c], pa); });
      static_for<2>([&](auto hh) {
        static_for<8>([&](auto i) {
          constexpr int r = 8 * hh + i;
          float p = fast_exp2(sa[r] * c2s);
          if constexpr (MASK) {
            const int iq = 16 * hh + 8 * kg + i;
            p = (iq >= lower && iq < upper) ? p : 0.f;
          }
          pf[r] = p;
          pb16[hh][int(i)] = static_cast<f16>(p);
        });
      });
      static_for<NT>([&](auto dt) {
        static_for<2>([&](auto c) {
          constexpr int at = S::Q_EL + 128 * c + 1024 * dt;
          ta[dt][c] = lds_tr16x2h(tp[0] + at, tp[1] + at);
        });
      });
      static_for<NC + 1>([&](auto i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, MASK ? 9 : 5, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, i < NC ? 2 : 0, 0);
      });
      };
      if (full) phase3(std::false_type{});
      else phase3(std::true_type{});
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (COPY) copy_part(std::integral_constant<int, 1>{});
      // (4) dV^T += dO^T P with dS = P (dP - D) on the VALU and the transpose
      // reads of Q^T
      f16x8 tq[NT][2];
      static_for<NT>([&](auto dt) {
        static_for<2>([&](auto c) { dva[dt] = mfma32h(ta[dt][c], pb16[c], dva[dt]); });
      });
      static_for<2>([&](auto hh) {
        static_for<8>([&](auto i) {
          constexpr int r = 8 * hh + i;
          db16[hh][int(i)] = static_cast<f16>(pf[r] * pa[r]);
        });
      });
      static_for<NT>([&](auto dt) {
        static_for<2>([&](auto c) {
          constexpr int at = 128 * c + 1024 * dt;
          tq[dt][c] = lds_tr16x2h(tp[0] + at, tp[1] + at);
        });
      });
      static_for<2 * NT>([&](auto i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (COPY) copy_part(std::integral_constant<int, 2>{});
      // (5) dK^T += Q^T dS
      static_for<NT>([&](auto dt) {
        static_for<2>([&](auto c) { dka[dt] = mfma32h(tq[dt][c], db16[c], dka[dt]); });
      });
    };

    // ---- compute a step of two heads: the products of one head run while the
    // VALU works on the other's scores, so that no product waits for them and
    // the matrix cores always have one queued.  Phases of NC + 1 or 2 NT
    // products each: S of head 0, S of head 1 (exp of head 0), dP of 0 (exp of
    // 1), dP of 1 (dS of 0), dV of 0 (dS of 1), dK of 0, dV of 1, dK of 1.  Each
    // operand is read AH products before the one that takes it, also across
    // phases.  Masks as in step().
    auto step2 = [&](bool full, const bf16 *Qs, int lower, int upper) {
      constexpr int NC = D / 16, NT = D / 32, AH = 4;
      constexpr int N1 = NC + 1, N2 = 2 * NT;   // products of an S / dP, a dV / dK phase
      constexpr int NOPS = 4 * N1 + 4 * N2;
      const bf16 *Ag = Qs + 2 * S::Q_EL + 8 * l;
      const bf16 *rp[2] = {Qs + qoff[0], Qs + qoff[1]};
      const f16 *tp[2] = {reinterpret_cast<const f16 *>(Qs) + troff[0],
                          reinterpret_cast<const f16 *>(Qs) + troff[1]};
      f32x16 sa[2], pa[2];        // S - LSE / scale, then P; dP - D
      f16x8 p16[2][2], s16[2][2];  // P and dS as operands
      f16x8 op[NOPS];
      // phase and product of operation n
      auto rd = [&](auto n_t) {
        constexpr int n = decltype(n_t)::value;
        if constexpr (n < 4 * N1) {
          constexpr int ph = n / N1, i = n % N1, hb = ph & 1, which = ph / 2;   // Q, then dO
          if constexpr (i == 0)
            op[n] = *reinterpret_cast<const f16x8 *>(Ag + hb * S::HEAD_EL + which * (kAugEl / 2));
          else
            op[n] = *reinterpret_cast<const f16x8 *>(rp[(i - 1) & 1] + hb * S::HEAD_EL +
                                                    which * S::Q_EL + 1024 * ((i - 1) >> 1));
        } else if constexpr (n < NOPS) {
          constexpr int m = n - 4 * N1, ph = m / N2, j = m % N2, hb = ph / 2;
          constexpr int dt = j >> 1, c = j & 1;
          constexpr int at = hb * S::HEAD_EL + (ph & 1 ? 0 : S::Q_EL) + 128 * c + 1024 * dt;
          op[n] = lds_tr16x2h(tp[0] + at, tp[1] + at);   // dO^T, then Q^T
        }
      };
      // VALU elements of head hb: P = exp2((S - LSE / scale) c2) and its rounding;
      // dS = P (dP - D) and its rounding.  Register 8 hh + i is row 16 hh + 8 kg + i
      auto exp_el = [&](auto hb, auto r_t) {
        constexpr int r = decltype(r_t)::value;
        float p = fast_exp2(sa[hb][r] * c2s);
        asm volatile("" : "+v"(p));   // stays in its slot
        sa[hb][r] = p;
      };
      auto mask = [&](auto hb) {
        int lo = lower - 8 * kg, hi = upper - 8 * kg;
        asm volatile("" : "+v"(lo), "+v"(hi));   // the comparisons stay in this branch
        static_for<16>([&](auto r) {
          constexpr int iq = 16 * (r >> 3) + (r & 7);
          sa[hb][int(r)] = (iq >= lo && iq < hi) ? sa[hb][int(r)] : -INFINITY;
        });
      };
      auto p_round = [&](auto hb, auto r_t) {
        constexpr int r = decltype(r_t)::value;
        p16[hb][r >> 3][r & 7] = static_cast<f16>(sa[hb][r]);
      };
      auto ds_el = [&](auto hb, auto r_t) {
        constexpr int r = decltype(r_t)::value;
        s16[hb][r >> 3][r & 7] = static_cast<f16>(sa[hb][r] * pa[hb][r]);
      };
      // 16 elements over the slots [2, n) of a phase of n products
      auto spread = [&](auto i_t, auto n_t, auto &&f) {
        constexpr int i = decltype(i_t)::value, n = decltype(n_t)::value;
        if constexpr (i >= 2) {
          constexpr int a = 16 * (i - 2) / (n - 2), b = 16 * (i - 1) / (n - 2);
          static_for<b - a>([&](auto e) { f(std::integral_constant<int, a + e>{}); });
        }
      };
      using H0 = std::integral_constant<int, 0>;
      using H1 = std::integral_constant<int, 1>;
      using L1 = std::integral_constant<int, N1>;
      using L2 = std::integral_constant<int, N2>;
      static_for<AH>([&](auto n) { rd(n); });
      __builtin_amdgcn_sched_barrier(0);
      static_for<4>([&](auto ph) {
        static_for<N1>([&](auto i) {
          constexpr int n = ph * N1 + i, hb = ph & 1;
          f32x16 &acc = ph < 2 ? sa[hb] : pa[hb];
          if constexpr (i == 0) acc = mfma32h(op[n], ones3, mfma_zero_c());
          else acc = mfma32h(op[n], ph < 2 ? kf[i > 0 ? i - 1 : 0] : vf[i > 0 ? i - 1 : 0], acc);
          rd(std::integral_constant<int, n + AH>{});
          if constexpr (ph == 1) spread(i, L1{}, [&](auto r) { exp_el(H0{}, r); });
          if constexpr (ph == 2) {
            if constexpr (i < 2)
              static_for<8>([&](auto e) { p_round(H0{}, std::integral_constant<int, 8 * i + e>{}); });
            spread(i, L1{}, [&](auto r) { exp_el(H1{}, r); });
          }
          if constexpr (ph == 3) {
            if constexpr (i < 2)
              static_for<8>([&](auto e) { p_round(H1{}, std::integral_constant<int, 8 * i + e>{}); });
            spread(i, L1{}, [&](auto r) { ds_el(H0{}, r); });
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (ph < 2)
          if (!full) mask(ph);
        if constexpr (ph == 1) copy_part(std::integral_constant<int, 0>{});
        if constexpr (ph == 3) copy_part(std::integral_constant<int, 1>{});
      });
      static_for<4>([&](auto ph) {
        static_for<N2>([&](auto j) {
          constexpr int n = 4 * N1 + ph * N2 + j, hb = ph / 2, dt = j >> 1, c = j & 1;
          if constexpr (ph & 1) dka[dt] = mfma32h(op[n], s16[hb][c], dka[dt]);
          else dva[dt] = mfma32h(op[n], p16[hb][c], dva[dt]);
          rd(std::integral_constant<int, n + AH>{});
          if constexpr (ph == 0) spread(j, L2{}, [&](auto r) { ds_el(H1{}, r); });
          __builtin_amdgcn_sched_barrier(0);
        });
        if constexpr (ph == 1) copy_part(std::integral_constant<int, 2>{});
      });
    };

    // Steps are walked once, at issue; what the compute side needs of the step
    // in ring stage j (lo | hi << 8 | two << 16, and the q_loc of the block's
    // row 0) waits in lane j of desc / desc_qb.
    StepIter iss{tiles, T, n_q, n_kv, key0, key0 + item.r0,
                 key0 + (item.r1 < len ? item.r1 : len), h_q, g, G, kloc0, 2 * S::HEAD_EL / 1024};
    iss.start();
    int desc = 0, desc_qb = 0;
    int issued = 0, computed = 0;
    // ring stage and descriptor of the next step to copy; after the last one,
    // its copies are repeated into the free stages, so that every iteration
    // posts as many and no product phase branches on it
    auto next_step = [&](int posted) {
      constexpr uint32_t bytes = 2u * S::STAGE_EL / kWaves;
      const int sg = posted & (S::NSTAGE - 1);
      cp_dst = lds_addr(smem + sg * S::STAGE_EL) + bytes * w;
      if (!iss.valid) return;
      cp_src = reinterpret_cast<const char *>(rec) + (uniform64(iss.rec) << 10) + bytes * w;
      if (l == sg) {
        desc = iss.lo() | iss.hi() << 8 | (iss.two() ? 1 << 16 : 0);
        desc_qb = iss.qb();
      }
      iss.next();
      ++issued;
    };
    if (iss.valid) {
      for (int i = 0; i < S::NSTAGE - 1; ++i) {
        next_step(i);
        copy_all();
      }
    }
    // one step per iteration; the loop of items whose every step has two heads
    // is one of its own (accumulators that merge from two bodies in each
    // iteration cost copies)
    auto steps = [&](auto pairs_t) {
      while (computed < issued) {
        // this step's copies are in; the two later steps' stay in flight
        wait_vm_n<(S::NSTAGE - 2) * S::LOADS>();
        barrier_nofence();
        // every wave is past the step before: the next one goes into its stage
        next_step(computed + S::NSTAGE - 1);

        const int sg = computed & (S::NSTAGE - 1);
        const int dsc = __builtin_amdgcn_readlane(desc, sg);
        const int lo_l = dsc & 0xff, hi_l = (dsc >> 8) & 0xff;
        const bool two = (dsc >> 16) != 0;
        const int qb = __builtin_amdgcn_readlane(desc_qb, sg);   // q_loc of the block's row 0
        if (kw0 <= qb + hi_l - 1) {
          const bf16 *Qs = smem + sg * S::STAGE_EL;
          // interior blocks: every row inside the fragment and at or after every key
          const bool full = lo_l == 0 && hi_l == kRows && wave_keys_ok && kw0 + 31 <= qb;
          const int need = kl - qb;                               // first iq with q_loc >= kl
          const int lower = need > lo_l ? (need < kRows ? need : kRows) : lo_l;
          const int upper = key_ok ? hi_l : 0;
          if constexpr (decltype(pairs_t)::value) {
            step2(full, Qs, lower, upper);
          } else {
            step(std::true_type{}, full, Qs, lower, upper);
            if (two) step(std::false_type{}, full, Qs + S::HEAD_EL, lower, upper);
          }
        } else {
          copy_all();
        }
        ++computed;
      }
    };
    if (odd_heads) {
      steps(std::false_type{});
    } else {
      // of four places modulo 32 bytes the best: 91.9 ms on the 256K share
      // against 92.5 to 92.6
      align_code<5>();
      steps(std::true_type{});
    }

    // ---- write dK, dV for this wave's 32 keys
    if (key_ok && item.slot >= 0) {
      // a part of a split item: unscaled fp32 dK and dV (key 32 w + ln)
      float *op = parts + (size_t)item.slot * 2 * fwd_part_floats(D) + (size_t)(32 * w + ln) * D +
                  8 * kg;
      static_for<D / 32>([&](auto dt) {
        static_for<4>([&](auto q4) {
          constexpr int at = 32 * dt + 16 * (q4 >> 1) + 4 * (q4 & 1), r0 = 4 * q4;
          *reinterpret_cast<float4 *>(op + at) = make_float4(
              dka[dt][r0], dka[dt][r0 + 1], dka[dt][r0 + 2], dka[dt][r0 + 3]);
          *reinterpret_cast<float4 *>(op + fwd_part_floats(D) + at) = make_float4(
              dva[dt][r0], dva[dt][r0 + 1], dva[dt][r0 + 2], dva[dt][r0 + 3]);
        });
      });
    } else if (key_ok) {
      const size_t base = ((size_t)krow * h_kv + g) * D + 8 * kg;
      static_for<D / 32>([&](auto dt) {
        static_for<2>([&](auto hh) {
          const size_t off = base + 32 * dt + 16 * hh;
          if (accumulate) {
            float4 *dkp = reinterpret_cast<float4 *>(static_cast<float *>(dk_out) + off);
            float4 *dvp = reinterpret_cast<float4 *>(static_cast<float *>(dv_out) + off);
            static_for<2>([&](auto e) {
              constexpr int r0 = 8 * hh + 4 * e;
              float4 a = dkp[e], bb = dvp[e];
              a.x += dka[dt][r0 + 0] * dk_mul; bb.x += dva[dt][r0 + 0] * dv_mul;
              a.y += dka[dt][r0 + 1] * dk_mul; bb.y += dva[dt][r0 + 1] * dv_mul;
              a.z += dka[dt][r0 + 2] * dk_mul; bb.z += dva[dt][r0 + 2] * dv_mul;
              a.w += dka[dt][r0 + 3] * dk_mul; bb.w += dva[dt][r0 + 3] * dv_mul;
              dkp[e] = a;
              dvp[e] = bb;
            });
          } else {
            bf16x8 a, bb;
            static_for<8>([&](auto i) {
              a[int(i)] = static_cast<bf16>(dka[dt][8 * hh + i] * dk_mul);
              bb[int(i)] = static_cast<bf16>(dva[dt][8 * hh + i] * dv_mul);
            });
            *reinterpret_cast<bf16x8 *>(static_cast<bf16 *>(dk_out) + off) = a;
            *reinterpret_cast<bf16x8 *>(static_cast<bf16 *>(dv_out) + off) = bb;
          }
        });
      });
    }
    wait_vm_n<0>();
    __syncthreads();   // the ring is reused by the next item
  }
}

// Sums the parts of every split dK / dV item (hdr[kBwdSplits] records) in row
// order and writes dK and dV as the kernel does for whole items.  Work shared
// as in fwd_combine_kernel (16 keys to a workgroup, 16 threads to a key).
template <int D>
__global__ __launch_bounds__(256) void bwd_dkdv_combine_kernel(
    const BwdSplit *__restrict__ splits, const int32_t *__restrict__ hdr,
    const float *__restrict__ parts, const int64_t *__restrict__ cu, int h_kv, float scale,
    void *__restrict__ dk_out, void *__restrict__ dv_out, int accumulate) {
  constexpr size_t PF = fwd_part_floats(D);
  constexpr int W = D / kCombineThreads;   // columns of a thread
  const int count = hdr[kBwdSplits] * kCombineSplit;
  const float s_q = fp16_scale((uint32_t)hdr[kMaxAbs + 0], false);
  const float s_o = fp16_scale((uint32_t)hdr[kMaxAbs + 1], true);
  const float s_v = fp16_scale((uint32_t)hdr[kMaxAbs + 3], true);
  const float mul[2] = {scale / (s_q * s_o * s_v), 1.f / s_o};   // as in the kernel
  const int tid = threadIdx.x, col = (tid % kCombineThreads) * W;
  for (int e = blockIdx.x; e < count; e += gridDim.x) {
    const BwdSplit sp = splits[e / kCombineSplit];
    const int kr = e % kCombineSplit * kCombineRows + tid / kCombineThreads;
    const int64_t key0 = cu[sp.item.sample], key = key0 + (int64_t)sp.item.kb * kBwdBK + kr;
    if (key >= cu[sp.item.sample + 1]) continue;
    const float *src = parts + (size_t)sp.base * 2 * PF + (size_t)kr * D + col;
    float acc[2][W];
#pragma unroll
    for (int i = 0; i < 2 * W; ++i) acc[i / W][i % W] = 0.f;
#pragma unroll 4
    for (int p = 0; p < sp.parts; ++p) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int i = 0; i < W / 4; ++i) {
          const float4 v = *reinterpret_cast<const float4 *>(src + (2 * p + x) * PF + 4 * i);
          acc[x][4 * i] += v.x;
          acc[x][4 * i + 1] += v.y;
          acc[x][4 * i + 2] += v.z;
          acc[x][4 * i + 3] += v.w;
        }
    }
    const size_t off = ((size_t)key * h_kv + sp.item.g) * D + col;
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      void *out = x ? dv_out : dk_out;
#pragma unroll
      for (int i = 0; i < W / 4; ++i) {
        if (accumulate) {
          float4 *op = reinterpret_cast<float4 *>(static_cast<float *>(out) + off) + i;
          float4 a = *op;
          a.x += acc[x][4 * i] * mul[x];
          a.y += acc[x][4 * i + 1] * mul[x];
          a.z += acc[x][4 * i + 2] * mul[x];
          a.w += acc[x][4 * i + 3] * mul[x];
          *op = a;
        } else {
          bf16x4 v;
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = static_cast<bf16>(acc[x][4 * i + j] * mul[x]);
          *reinterpret_cast<bf16x4 *>(static_cast<bf16 *>(out) + off + 4 * i) = v;
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
static size_t align256b(size_t x) { return (x + 255) / 256 * 256; }

BwdLayout bwd_layout(int64_t T, int64_t n, int64_t n_q, int64_t n_kv, int h_q, int h_kv, int d) {
  BwdLayout L;
  // a split item's parts take its place: kBwdSplitSlots of them at most
  L.max_blocks = (n_kv / kBwdBK + n + 1) * (int64_t)h_kv;
  L.max_items = L.max_blocks + kBwdSplitSlots;
  L.max_qitems = fwd_max_items(T, n, n_q, h_q, h_kv);
  L.nq_pad = (n_q + kRows - 1) / kRows * kRows;
  L.hdr = 0;
  L.ext = kHdrBytes;
  L.gmask = align256b(L.ext + (size_t)n * sizeof(int32_t));
  L.items = align256b(L.gmask + (size_t)n * sizeof(unsigned long long));
  L.qitems = align256b(L.items + (size_t)L.max_items * sizeof(BwdItem));
  L.rec = align256b(L.qitems + (size_t)L.max_qitems * sizeof(FwdItem));
  // one record more: a step of one head copies the record after its own
  L.k16 = align256b(L.rec + (size_t)(L.nq_pad / kRows * h_q + 1) * rec_els(d) * sizeof(f16));
  L.v16 = align256b(L.k16 + (size_t)n_kv * h_kv * d * sizeof(f16));
  L.stats = align256b(L.v16 + (size_t)n_kv * h_kv * d * sizeof(f16));
  L.splits = align256b(L.stats + (size_t)h_q * L.nq_pad * 2 * sizeof(float));
  L.max_parts = kFwdSplitSlots;
  L.bsplits = align256b(L.splits + (size_t)(L.max_parts / 2) * sizeof(FwdSplit));
  L.cov = align256b(L.bsplits + (size_t)(kBwdSplitSlots / 2) * sizeof(BwdSplit));
  // the partial slots serve the dQ kernel, then the dK / dV kernel
  L.parts = align256b(L.cov + (size_t)L.max_blocks * 2 * sizeof(int32_t));
  L.total = align256b(L.parts + (size_t)L.max_parts * fwd_part_floats(d) * sizeof(float));
  return L;
}

template <int D>
static int launch_bwd_d(const bf16 *q, const bf16 *k, const bf16 *v, const bf16 *o,
                        const float *lse, const bf16 *dout, const int64_t *cu, int64_t n,
                        const libra_tile_t *tiles, int64_t T, int64_t n_q, int64_t n_kv, int h_q,
                        int h_kv, float scale, bf16 *dq, void *dk, void *dv, bool accumulate,
                        char *ws, const BwdLayout &L, hipStream_t st, const KernelTimer *tm_kv,
                        const KernelTimer *tm_q) {
  int32_t *hdr = reinterpret_cast<int32_t *>(ws + L.hdr);
  int32_t *ext = reinterpret_cast<int32_t *>(ws + L.ext);
  auto *gmask = reinterpret_cast<unsigned long long *>(ws + L.gmask);
  BwdItem *items = reinterpret_cast<BwdItem *>(ws + L.items);
  FwdItem *qitems = reinterpret_cast<FwdItem *>(ws + L.qitems);
  f16 *rec = reinterpret_cast<f16 *>(ws + L.rec);
  f16 *k16 = reinterpret_cast<f16 *>(ws + L.k16);
  f16 *v16 = reinterpret_cast<f16 *>(ws + L.v16);
  float *stats = reinterpret_cast<float *>(ws + L.stats);
  int32_t *cov = reinterpret_cast<int32_t *>(ws + L.cov);
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_bwd_dkdv_kernel<D>),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)KvShape<D>::SMEM) != hipSuccess)
      return fail(LIBRA_EHIP, "hipFuncSetAttribute failed");
    attr_set = true;
  }
  // bf16 dK / dV are written where a covered row attends and zero elsewhere
  const int64_t n16 = accumulate ? 0 : n_kv * h_kv * D * (int64_t)sizeof(bf16) / 16;
  const unsigned zero_blocks = (unsigned)std::min<int64_t>((n16 + 255) / 256, 4096);
  if (T == 0 && n16 > 0) {
    hipLaunchKernelGGL(zero_kernel, dim3(zero_blocks), dim3(256), 0, st, static_cast<uint4 *>(dk),
                       n16);
    hipLaunchKernelGGL(zero_kernel, dim3(zero_blocks), dim3(256), 0, st, static_cast<uint4 *>(dv),
                       n16);
  }
  if (T > 0) {
    int dev = 0, cus = 256;
    hipGetDevice(&dev);
    hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    // the dQ kernel runs one workgroup per CU; its items split K like the
    // forward's when there are few of them, but only when whole rounds of items
    // would leave workgroups idle: measured on calls of one tile, splitting
    // items that already fill the grid cost dQ 2-4%, while the forward gained
    // 3-5% from it
    auto *splits = reinterpret_cast<FwdSplit *>(ws + L.splits);
    float *parts = reinterpret_cast<float *>(ws + L.parts);
    const int max_parts = may_split(n_kv) ? L.max_parts : 0;
    hipLaunchKernelGGL(prep_bwd_kernel, dim3(2), dim3(kPrepThreads), 0, st,
                       BwdPrep{cu, n, tiles, T, h_q, h_kv, n_q, n_kv, hdr, ext, gmask, items,
                               L.max_items, cus, reinterpret_cast<BwdSplit *>(ws + L.bsplits), cov,
                               cov + L.max_blocks},
                       FwdPrep{cu, n, tiles, T, h_q, h_kv, n_q, n_kv, hdr, qitems, L.max_qitems, 0,
                               cus, cus, max_parts, 1, splits});
    // K and V rows: at least eight for a wave (every workgroup that finds a new
    // maximum posts an atomic on the same two slots: 2048 of them took 24 us on
    // 4096 rows)
    const unsigned kv_blocks =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>((n_kv + 31) / 32, (int64_t)cus * 8));
    const BwdPass pass{q, k, v, o, dout, lse, cu, n, tiles, h_q, h_kv, n_q, n_kv, L.nq_pad, scale,
                       hdr, ext, rec, k16, v16, stats, static_cast<uint4 *>(dk),
                       static_cast<uint4 *>(dv), n16, (unsigned)(T * kTileSplit), kv_blocks,
                       2 * zero_blocks};
    hipLaunchKernelGGL(bwd_max_kernel<D>,
                       dim3(pass.kv_blocks + pass.tile_blocks + pass.zero_blocks), dim3(256), 0,
                       st, pass);
    hipLaunchKernelGGL(bwd_copy_kernel<D>, dim3(pass.kv_blocks + pass.tile_blocks), dim3(256), 0,
                       st, pass);
    // dQ first: it writes the -D records the dK / dV kernel reads
    const int rc = launch_bwd_dq(D, q, dout, k, v, stats, cu, qitems, hdr, h_q, h_kv, n_q, n_kv,
                                 L.nq_pad, scale, dq, rec, splits, parts, max_parts, cus,
                                 st, tm_q);
    if (rc != LIBRA_OK) return rc;
    if (tm_kv) hipEventRecord(tm_kv->begin, st);
    hipLaunchKernelGGL(attn_bwd_dkdv_kernel<D>, dim3(cus), dim3(kThreads), KvShape<D>::SMEM, st,
                       k16, v16, rec, cu, tiles, T, items, hdr, h_q, h_kv, n_q, n_kv, scale,
                       scale * kLog2e, dk, dv, accumulate ? 1 : 0, parts);
    if (may_split_rows(n_kv))
      hipLaunchKernelGGL(bwd_dkdv_combine_kernel<D>, dim3(cus * 4), dim3(256), 0, st,
                         reinterpret_cast<const BwdSplit *>(ws + L.bsplits), hdr, parts, cu, h_kv,
                         scale, dk, dv, accumulate ? 1 : 0);
    if (tm_kv) hipEventRecord(tm_kv->end, st);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LIBRA_EHIP, "backward launch failed: %s", hipGetErrorString(e));
  return LIBRA_OK;
}

int launch_bwd(const void *q, const void *k, const void *v, const void *o, const float *lse,
               const void *dout, const int64_t *cu, int64_t n, const libra_tile_t *tiles,
               int64_t T, int64_t n_q, int64_t n_kv, int h_q, int h_kv, int d, float scale,
               void *dq, void *dk, void *dv, bool accumulate, void *ws, const BwdLayout &L,
               hipStream_t st, const KernelTimer *tm_kv, const KernelTimer *tm_q) {
  auto Q = static_cast<const bf16 *>(q);
  auto K = static_cast<const bf16 *>(k);
  auto V = static_cast<const bf16 *>(v);
  auto O = static_cast<const bf16 *>(o);
  auto dO = static_cast<const bf16 *>(dout);
  auto dQ = static_cast<bf16 *>(dq);
  char *W = static_cast<char *>(ws);
  if (d == 128)
    return launch_bwd_d<128>(Q, K, V, O, lse, dO, cu, n, tiles, T, n_q, n_kv, h_q, h_kv, scale,
                             dQ, dk, dv, accumulate, W, L, st, tm_kv, tm_q);
  return launch_bwd_d<64>(Q, K, V, O, lse, dO, cu, n, tiles, T, n_q, n_kv, h_q, h_kv, scale, dQ,
                          dk, dv, accumulate, W, L, st, tm_kv, tm_q);
}

}  // namespace libra
