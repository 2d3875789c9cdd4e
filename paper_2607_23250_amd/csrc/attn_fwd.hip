// Forward pass of document-masked causal attention over SH-Tiles (gfx950).
//
// What is computed: Eq. 1 of the paper under the block-diagonal causal mask of
// packing (Sec. 2.3), for the (row, query head) pairs covered by a list of
// SH-Tiles (Sec. 4.3.1).  Each tile is cut into work items on the device; a
// persistent kernel walks the items longest-first.
//
// Kernel structure (one work item = up to 4 query heads of one KV group x 32
// rows per head, or fewer heads x more rows; 4 waves, one (head, 32 rows) each):
//   * K and V blocks of 64 keys are staged in LDS as rows, double-buffered;
//     blocks are anchored at the sample start and only the row's own sample
//     is visited, so cross-document blocks are never touched.
//   * S^T = K Q^T with v_mfma_f32_32x32x16_bf16 (keys on M, queries on N), so
//     that every lane owns one query: the row max / row sum of the online
//     softmax are 32 in-lane values plus one exchange with lane ^ 32.
//   * O^T += V^T P^T with the same instruction; P^T comes straight from the
//     S^T accumulators (bf16), V^T from the row-major V tile through the LDS
//     transpose reads.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "attn_common.h"
#include "attn_items.h"
#include "errors.h"

namespace libra {

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kPrepThreads) void prep_fwd_kernel(FwdPrep a) {
  __shared__ FwdPrepLds lds;
  prep_fwd(a, lds);
}

// Merges the parts of every split item (hdr[kFwdSplits] records): per row,
// m = max_p m_p, l = sum_p l_p 2^(m_p - m), O = sum_p O_p 2^(m_p - m) / l and
// LSE = (m + log2 l) ln 2, the online-softmax recurrence applied across the
// key ranges.  Bound by the reads of the parts; an item is shared by
// kCombineSplit workgroups of 16 rows, 16 threads to a row: with one workgroup
// per item and two threads to a row, a call of one tile (2048 rows x 4 heads,
// 64 items of 25 parts) kept 64 CUs busy with one chain of loads each, and
// took 113 us; forward and merge together 865 us, now 778.
template <int D>
__global__ __launch_bounds__(256) void fwd_combine_kernel(
    const FwdSplit *__restrict__ splits, const int32_t *__restrict__ hdr,
    const float *__restrict__ parts, int h_q, int64_t n_q, bf16 *__restrict__ o,
    float *__restrict__ lse) {
  constexpr size_t PF = fwd_part_floats(D);
  constexpr int W = D / kCombineThreads;   // columns of a thread
  const int count = hdr[kFwdSplits] * kCombineSplit;
  const int tid = threadIdx.x, col = (tid % kCombineThreads) * W;
  for (int e = blockIdx.x; e < count; e += gridDim.x) {
    const FwdSplit sp = splits[e / kCombineSplit];
    const int pr = e % kCombineSplit * kCombineRows + tid / kCombineThreads;
    const int w = pr >> 5, r = pr & 31;   // wave slice and row of the item
    const FwdItem &it = sp.item;
    const int wrow0 = (w / it.nh) * kRows;
    const int wrows = min(max(it.nrows - wrow0, 0), kRows);
    if (r >= wrows) continue;
    const int head = it.head0 + (w % it.nh);
    const int64_t row = (int64_t)it.q_row0 + wrow0 + r;
    const float *rec = parts + (size_t)sp.base * PF;
    float m = -INFINITY;
#pragma unroll 8
    for (int p = 0; p < sp.parts; ++p) m = fmaxf(m, rec[p * PF + (size_t)kFwdPartRows * D + pr]);
    float l = 0.f;
    float acc[W];
#pragma unroll
    for (int i = 0; i < W; ++i) acc[i] = 0.f;
#pragma unroll 4
    for (int p = 0; p < sp.parts; ++p) {
      const float *pt = rec + p * PF;
      const float mp = pt[(size_t)kFwdPartRows * D + pr];
      const float wgt = mp == -INFINITY ? 0.f : fast_exp2(mp - m);
      l += wgt * pt[(size_t)kFwdPartRows * D + kFwdPartRows + pr];
      const float4 *src = reinterpret_cast<const float4 *>(pt + (size_t)pr * D + col);
#pragma unroll
      for (int i = 0; i < W / 4; ++i) {
        const float4 x = src[i];
        acc[4 * i] += wgt * x.x;
        acc[4 * i + 1] += wgt * x.y;
        acc[4 * i + 2] += wgt * x.z;
        acc[4 * i + 3] += wgt * x.w;
      }
    }
    const float inv = 1.f / l;
    bf16 *op = o + ((size_t)row * h_q + head) * D + col;
#pragma unroll
    for (int i = 0; i < W / 4; ++i) {
      bf16x4 ov;
#pragma unroll
      for (int j = 0; j < 4; ++j) ov[j] = static_cast<bf16>(acc[4 * i + j] * inv);
      *reinterpret_cast<bf16x4 *>(op + 4 * i) = ov;
    }
    if (col == 0) lse[(size_t)head * n_q + row] = (m + __builtin_amdgcn_logf(l)) * kLn2;
  }
}

// ---------------------------------------------------------------------------
template <int D>
struct FwdShape {
  static constexpr int KC = D / 8;            // 16-byte columns of a K / V row
  static constexpr int K_EL = kFwdBN * D;
  static constexpr int STAGE = 2 * K_EL;      // K and V rows of one key block
  static constexpr int NK = kFwdBN * KC / 64 / kWaves;   // wave loads of 1 KB per tile
  static constexpr size_t SMEM = 2 * STAGE * sizeof(bf16);
};

// Workgroups per CU: at d = 64 the registers of three fit (12 heads, 20K
// tokens: 382 us against 422 with two; 131072 items of one key block: 1.63 ms
// against 1.88).  Which calls split items does not depend on it.
template <int D>
constexpr int kFwdPerCu = D == 64 ? 3 : 2;

template <int D>
__global__ __launch_bounds__(kThreads, kFwdPerCu<D>) void attn_fwd_kernel(
    const bf16 *__restrict__ q, const bf16 *__restrict__ k, const bf16 *__restrict__ v,
    const int64_t *__restrict__ cu, const FwdItem *__restrict__ items, int32_t *__restrict__ hdr,
    int h_q, int h_kv, int64_t n_q, int64_t n_kv, float c2,
    bf16 *__restrict__ o, float *__restrict__ lse, float *__restrict__ parts) {
  using S = FwdShape<D>;
  extern __shared__ __attribute__((aligned(16))) bf16 smem[];
  __shared__ int32_t s_item;
  const int tid = threadIdx.x, l = tid & 63, ln = l & 31, kg = l >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave index (uniform)
  const int q_serve = xcd_of_workgroup();
  int q_state = kTakeFirst;
  // per-lane LDS offsets (elements) of the operand reads, fixed for the kernel:
  // K rows perm32(ln) for S^T (chunk 2 c + kg: one offset per parity of c, then
  // 4 chunks per 2 steps of c), and the transpose reads of the V tile for the
  // V^T operand of O^T (rows = keys, as in the dQ kernel's K^T; one offset per
  // half, then 4 chunks per step of dt)
  constexpr int STEP4 = S::KC == 16 ? 128 : 256;   // elements from chunk j to chunk j + 4
  const int prow = perm32(ln);
  const int koff[2] = {swu<S::KC>(prow, kg), swu<S::KC>(prow, 2 + kg)};
  int troff[2];
  {
    const int grp = l >> 4, i = (l & 15) >> 2, r = l & 3;
    static_for<2>([&](auto hf) {
      troff[hf] = swu<S::KC>(8 * (grp >> 1) + 4 * hf + i, 2 * (grp & 1) + (r & 1)) + 4 * (r >> 1);
    });
  }
  // staging: wave load u fills unit w + 4 u of a tile; k_lane[u] is the lane's
  // byte offset from the block's first K (V) row
  uint32_t k_lane[S::NK];
  static_for<S::NK>([&](auto u) {
    const int wl = w + kWaves * u;
    k_lane[u] = 2u * (uint32_t)(swu_row<S::KC>(wl, l) * h_kv * D + 8 * swu_col<S::KC>(wl, l));
  });

  for (;;) {
    if (w == 0) {
      const int got = take_item(hdr, kFwdQ, q_serve, q_state);
      if (tid == 0) s_item = got;
    }
    __syncthreads();
    const int idx = __builtin_amdgcn_readfirstlane(s_item);
    if (idx < 0) break;
    const FwdItem it = items[idx];
    const int64_t key0 = cu[it.sample];
    const int head = it.head0 + (w % it.nh);
    const int wrow0 = (w / it.nh) * kRows;
    const int wrows = min(max(it.nrows - wrow0, 0), kRows);
    const bool active = wrows > 0;
    const int my_r = active ? min(ln, wrows - 1) : 0;
    const int64_t row = (int64_t)it.q_row0 + wrow0 + my_r;
    const int qloc = it.q_loc0 + wrow0 + my_r;
    const int wave_qmin = it.q_loc0 + wrow0;
    const int kb0 = it.kb0, nkb = it.kb1;   // key blocks [kb0, nkb)
    const int wave_nkb = active ? (it.q_loc0 + wrow0 + wrows - 1) / kFwdBN + 1 : 0;

    bf16x8 qf[D / 16];
    if (active) {
      const bf16 *qp = q + ((size_t)row * h_q + head) * D + 8 * kg;
      static_for<D / 16>([&](auto c) { qf[c] = *reinterpret_cast<const bf16x8 *>(qp + 16 * c); });
    }
    f32x16 oacc[D / 32];
    static_for<D / 32>([&](auto dt) { static_for<16>([&](auto r) { oacc[dt][int(r)] = 0.f; }); });
    float m_run = -INFINITY, l_run = 0.f;

    // global -> LDS, asynchronous: the K (part 0) or V (part 1) rows of key
    // block b (keys past the buffer read the last key instead; keys past the
    // row are masked, and their V rows meet P = 0)
    auto issue = [&](int b, int buf, int part) {
      const bf16 *src = part ? v : k;
      bf16 *dst = smem + buf * S::STAGE + part * S::K_EL;
      const int64_t kbase = key0 + (int64_t)b * kFwdBN;
      if (kbase + kFwdBN <= n_kv) {
        // whole block inside the buffer: one SGPR base, fixed per-lane offsets;
        // wave load u lands 1 KiB x (w + kWaves u) into the tile
        const bf16 *base = src + ((size_t)kbase * h_kv + it.g) * D;
        const uint32_t ld = lds_addr(dst) + 1024u * w;
        static_for<S::NK / 4>([&](auto h) {
          constexpr uint32_t d = 4 * h * kWaves * 1024u, e = kWaves * 1024u;
          g2l16x4r(base, k_lane[4 * h], k_lane[4 * h + 1], k_lane[4 * h + 2], k_lane[4 * h + 3],
                   ld + d, ld + d + e, ld + d + 2 * e, ld + d + 3 * e);
        });
        static_for<S::NK % 4>([&](auto i) {
          constexpr int u = S::NK / 4 * 4 + i;
          g2l16s(base, k_lane[u], ld + u * kWaves * 1024u);
        });
        return;
      }
      // the last block of the buffer: keys past it read the last key (masked)
      static_for<S::NK>([&](auto u) {
        const int wl = w + kWaves * u;
        const int col = swu_col<S::KC>(wl, l);
        int64_t key = key0 + (int64_t)b * kFwdBN + swu_row<S::KC>(wl, l);
        key = key < n_kv ? key : n_kv - 1;
        g2l16(src + ((size_t)key * h_kv + it.g) * D + 8 * col, dst + wl * 512);
      });
    };

    issue(kb0, 0, 0);
    issue(kb0, 0, 1);
    wait_vm_known();   // also Q: no wait for it inside the loop
    __syncthreads();
    for (int b = kb0; b < nkb; ++b) {
      const int buf = (b - kb0) & 1;
      // the next block's K rows after this block's S^T products, its V rows
      // after the softmax (the other workgroup on the CU keeps the matrix
      // cores busy while this one waits to issue; waves without rows in this
      // block post both at once)
      const bool more = b + 1 < nkb;
      if (b >= wave_nkb && more) {
        issue(b + 1, buf ^ 1, 0);
        issue(b + 1, buf ^ 1, 1);
      }
      if (b < wave_nkb) {
        constexpr int NC = D / 16, NT = D / 32, AHEAD = 4;
        const bf16 *Ks = smem + buf * S::STAGE;
        const bf16 *Vs = Ks + S::K_EL;
        // S^T: every operand is read AHEAD products before the one that takes
        // it.  Left to itself the compiler reads many of them right before
        // their product and waits for the LDS round trip, as often as 32 times
        // per block.  On the 1M share: 430 ms, 420 with the reads ahead here
        // and in O^T, 413 with the swu places too (1167 of the 1560 TFLOP/s
        // that a large matrix product reaches); at 32K tokens 3.18, 3.07, 3.06.
        f32x16 s[2];
        bf16x8 kop[2 * NC];   // product i: key tile i / NC, chunk i % NC
        const bf16 *kp[2] = {Ks + koff[0], Ks + koff[1]};
        auto rd = [&](auto i) {
          constexpr int t = i / NC, c = i % NC;
          kop[i] = *reinterpret_cast<const bf16x8 *>(kp[c & 1] + 32 * t * D + (c >> 1) * STEP4);
        };
        static_for<AHEAD>([&](auto i) { rd(i); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<2 * NC>([&](auto i) {
          constexpr int t = i / NC, c = i % NC;
          if constexpr (c == 0) static_for<16>([&](auto r) { s[t][int(r)] = 0.f; });
          s[t] = mfma32(kop[i], qf[c], s[t]);
          if constexpr (i + AHEAD < 2 * NC) rd(std::integral_constant<int, i + AHEAD>{});
          __builtin_amdgcn_sched_barrier(0);
        });
        if (more) issue(b + 1, buf ^ 1, 0);
        // keys past the row are masked only in blocks that reach past the
        // wave's first row (the diagonal block of each row)
        if (b * kFwdBN + kFwdBN - 1 > wave_qmin) {
          static_for<2>([&](auto t) {
            static_for<16>([&](auto r) {
              const int kl = b * kFwdBN + 32 * t + 16 * (r >> 3) + 8 * kg + (r & 7);
              if (kl > qloc) s[t][int(r)] = -INFINITY;
            });
          });
        }
        // P with the running max.  The block's row sum of P (needed anyway)
        // bounds every P of the row, so the running max only has to move
        // when that sum exceeds 256 (every P then stays <= 256, as with a
        // max test); the first block always sets it.  Only then is the
        // block's row max computed, the row rescaled and P recomputed.
        bf16x8 pf[4];
        float ps = 0.f;
        auto expo = [&](float neg_m) {
          ps = 0.f;
          static_for<2>([&](auto t) {
            static_for<16>([&](auto r) {
              const float p = fast_exp2(__builtin_fmaf(s[t][int(r)], c2, neg_m));
              ps += p;
              pf[2 * t + (r >> 3)][r & 7] = static_cast<bf16>(p);
            });
          });
        };
        bool move = true;
        if (b > kb0) {
          expo(-m_run);
          move = !(row_sum2(ps) <= 256.f);
        }
        if (__builtin_amdgcn_ballot_w64(move)) {
          float mx = -INFINITY;
          static_for<2>([&](auto t) {
            static_for<16>([&](auto r) { mx = fmaxf(mx, s[t][int(r)]); });
          });
          mx = row_max2(mx) * c2;
          const float alpha = move ? fast_exp2(m_run - mx) : 1.f;
          m_run = move ? mx : m_run;
          l_run *= alpha;
          static_for<D / 32>([&](auto dt) {
            static_for<16>([&](auto r) { oacc[dt][int(r)] *= alpha; });
          });
          expo(-m_run);
        }
        l_run += ps;
        constexpr int TA = 4;
        bf16x8 vop[4 * NT];
        const bf16 *vp[2] = {Vs + troff[0], Vs + troff[1]};
        auto rt = [&](auto j) {
          constexpr int at = 16 * D * (j / NT) + STEP4 * (j % NT);
          vop[j] = lds_tr16x2(vp[0] + at, vp[1] + at);
        };
        static_for<TA>([&](auto j) { rt(j); });
        if (more) issue(b + 1, buf ^ 1, 1);
        __builtin_amdgcn_sched_barrier(0);
        // O^T += V^T P^T; product j takes key chunk j / NT (16 keys from tile
        // row 16 j / NT), 32 columns j % NT, its operand read TA products ahead
        static_for<4 * NT>([&](auto j) {
          oacc[j % NT] = mfma32(vop[j], pf[j / NT], oacc[j % NT]);
          if constexpr (j + TA < 4 * NT) rt(std::integral_constant<int, j + TA>{});
          __builtin_amdgcn_sched_barrier(0);
        });
      }
      wait_vm();
      __syncthreads();
    }

    if (active && it.slot >= 0) {
      // a part of a split item: unnormalised O, the running max and the row
      // sum into its partial slot (rows w * 32 + ln), merged by
      // fwd_combine_kernel
      const float l_tot = row_sum2(l_run);
      if (ln < wrows) {
        float *rec = parts + (size_t)it.slot * fwd_part_floats(D);
        float *op = rec + (size_t)(w * kRows + ln) * D + 8 * kg;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            float4 *dst = reinterpret_cast<float4 *>(op + 32 * dt + 16 * hh);
            dst[0] = make_float4(oacc[dt][8 * hh], oacc[dt][8 * hh + 1], oacc[dt][8 * hh + 2],
                                 oacc[dt][8 * hh + 3]);
            dst[1] = make_float4(oacc[dt][8 * hh + 4], oacc[dt][8 * hh + 5],
                                 oacc[dt][8 * hh + 6], oacc[dt][8 * hh + 7]);
          }
        if (kg == 0) {
          rec[(size_t)kFwdPartRows * D + w * kRows + ln] = m_run;
          rec[(size_t)kFwdPartRows * D + kFwdPartRows + w * kRows + ln] = l_tot;
        }
      }
    } else if (active) {
      const float l_tot = row_sum2(l_run);
      const float inv = 1.f / l_tot;
      if (ln < wrows) {
        bf16 *op = o + ((size_t)row * h_q + head) * D + 8 * kg;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            bf16x8 ov;
#pragma unroll
            for (int i = 0; i < 8; ++i) ov[i] = static_cast<bf16>(oacc[dt][8 * hh + i] * inv);
            *reinterpret_cast<bf16x8 *>(op + 32 * dt + 16 * hh) = ov;
          }
        if (kg == 0) lse[(size_t)head * n_q + row] = (m_run + __builtin_amdgcn_logf(l_tot)) * kLn2;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Host launcher.  `ws` is laid out as: header | items.
static size_t align256(size_t x) { return (x + 255) / 256 * 256; }

int64_t fwd_max_items(int64_t T, int64_t n, int64_t n_q, int h_q, int h_kv) {
  // items <= rows*heads/64 (an item covers >= 64 (row, head) pairs or ends a
  // fragment) + fragments * head chunks.
  // A split item's parts take its place: kFwdSplitSlots of them at most.
  const int64_t frags = T + (int64_t)h_q * n;
  return n_q * (int64_t)h_q / 64 + frags * (int64_t)(h_kv + h_q / 4 + 1) + 1 + kFwdSplitSlots;
}

FwdLayout fwd_layout(int64_t T, int64_t n, int64_t n_q, int64_t n_kv, int h_q, int h_kv, int d,
                     bool split) {
  FwdLayout L;
  L.max_items = fwd_max_items(T, n, n_q, h_q, h_kv);
  L.hdr = 0;
  L.items = kHdrBytes;
  L.splits = align256(L.items + (size_t)L.max_items * sizeof(FwdItem));
  L.max_parts = split ? kFwdSplitSlots : 0;
  // a split item has at least two parts
  L.parts = align256(L.splits + (size_t)(L.max_parts / 2) * sizeof(FwdSplit));
  L.total = align256(L.parts + (size_t)L.max_parts * fwd_part_floats(d) * sizeof(float));
  return L;
}

template <int D>
static int launch_fwd_d(const bf16 *q, const bf16 *k, const bf16 *v, const int64_t *cu,
                        int64_t n, const libra_tile_t *tiles, int64_t T, int64_t n_q,
                        int64_t n_kv, int h_q, int h_kv, float scale, bf16 *o, float *lse,
                        char *ws, const FwdLayout &L, hipStream_t st, const KernelTimer *tm) {
  int32_t *hdr = reinterpret_cast<int32_t *>(ws + L.hdr);
  FwdItem *items = reinterpret_cast<FwdItem *>(ws + L.items);
  auto *splits = reinterpret_cast<FwdSplit *>(ws + L.splits);
  float *parts = reinterpret_cast<float *>(ws + L.parts);
  static bool attr_set = false;
  if (!attr_set) {
    if (hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_fwd_kernel<D>),
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)FwdShape<D>::SMEM) != hipSuccess)
      return fail(LIBRA_EHIP, "hipFuncSetAttribute failed");
    attr_set = true;
  }
  int dev = 0, cus = 256;
  hipGetDevice(&dev);
  hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const int grid = cus * kFwdPerCu<D>;
  const int max_parts = may_split(n_kv) ? L.max_parts : 0;
  hipLaunchKernelGGL(prep_fwd_kernel, dim3(1), dim3(kPrepThreads), 0, st,
                     FwdPrep{cu, n, tiles, T, h_q, h_kv, n_q, n_kv, hdr, items, L.max_items, 1,
                             grid, cus * 2, max_parts, 0, splits});
  if (tm) hipEventRecord(tm->begin, st);
  hipLaunchKernelGGL(attn_fwd_kernel<D>, dim3(grid), dim3(kThreads), FwdShape<D>::SMEM, st, q,
                     k, v, cu, items, hdr, h_q, h_kv, n_q, n_kv, scale * kLog2e, o,
                     lse, parts);
  if (max_parts > 0)
    hipLaunchKernelGGL(fwd_combine_kernel<D>, dim3(cus * 4), dim3(256), 0, st, splits, hdr, parts,
                       h_q, n_q, o, lse);
  if (tm) hipEventRecord(tm->end, st);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(LIBRA_EHIP, "forward launch failed: %s", hipGetErrorString(e));
  return LIBRA_OK;
}

int launch_fwd(const void *q, const void *k, const void *v, const int64_t *cu, int64_t n,
               const libra_tile_t *tiles, int64_t T, int64_t n_q, int64_t n_kv, int h_q,
               int h_kv, int d, float scale, void *o, float *lse, void *ws,
               const FwdLayout &L, hipStream_t st, const KernelTimer *tm) {
  auto Q = static_cast<const bf16 *>(q);
  auto K = static_cast<const bf16 *>(k);
  auto V = static_cast<const bf16 *>(v);
  auto O = static_cast<bf16 *>(o);
  char *W = static_cast<char *>(ws);
  if (d == 128)
    return launch_fwd_d<128>(Q, K, V, cu, n, tiles, T, n_q, n_kv, h_q, h_kv, scale, O, lse, W, L,
                             st, tm);
  return launch_fwd_d<64>(Q, K, V, cu, n, tiles, T, n_q, n_kv, h_q, h_kv, scale, O, lse, W, L, st,
                          tm);
}

}  // namespace libra
