// Launch plan of heart_block_sparse_attn: which XCD walks which heads, and in which order the
// rows (query blocks) of a head start.  Layout: heart_internal.h.
//
// One launch; no workgroup needs what another one writes:
//   near_order   (one workgroup per head, if the workspace has room) rows in batches of similar
//                kept lists, the sequence the attention then follows
//   plan_heads   (one workgroup) total kept count per head, heads ranked by it and assigned
//                greedily to the XCDs, head table, cursors; beyond 1024 heads they are dealt to the XCDs
//                without a look at the totals, which class_order then writes (one workgroup
//                that sums them all up takes longer than the others together: 131072 heads of
//                one row, whole call 3069 -> 2805 us)
//   class_order  (one workgroup per head, up to 2^20) rows by count class, longest first: the sequence of a
//                workspace without room for the other (it is there in every plan)
// Bound by latency.  At 40 heads of 256 rows 14 us without near_order and 15 to 22 with it (longer between long
// attention launches, at the clock these leave), at 24 heads of 931 rows 13 and 87 to 124.
#include "heart_internal.h"

namespace heart {

namespace {

constexpr int kOrderClasses = 32;   // count classes of the per-head sort
constexpr int kPlanMaxHeads = 1024; // beyond this heads are dealt to the XCDs round-robin
constexpr int kPlanThreads = 1024;
constexpr int kOrderCols = 256;     // columns of the class histogram
constexpr int kPlanMaxGroups = 1 << 20;  // workgroups per part of the launch (a launch has less than 2^32 threads)
static_assert(kCursorSpread * kNumXcd * sizeof(int) + kCursorLine <= kCursorBytes, "room of the spread cursors");

// kept count of a row as the attention kernel reads it
__device__ __forceinline__ int row_count(const int *kept_count, int i, int Nb) {
  return min(max(kept_count[i], 0), Nb);
}

// Heads ranked by total kept count, greedy assignment of heads (heaviest first) to the least
// loaded XCD, head table, cursors (`spread` if given, else the header's) reset behind the items that the
// n_wg attention workgroups start with.
template <int kThreads>
__device__ __forceinline__ void plan_heads(const int *__restrict__ kept_count, int BH, int Nb, int n_wg, int n_few,
                                           int *__restrict__ plan, int *__restrict__ spread, unsigned char *lds) {
  int *w_head = reinterpret_cast<int *>(lds);
  int *sorted = w_head + kPlanMaxHeads, *xcd_of = sorted + kPlanMaxHeads, *rank_of = xcd_of + kPlanMaxHeads;
  __shared__ int n_heads[kNumXcd], off[kNumXcd];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (BH <= kPlanMaxHeads) {
    for (int bh = wave; bh < BH; bh += kThreads / 64) {
      int w = 0;
#pragma unroll 8
      for (int i = lane; i < Nb; i += 64) w += row_count(kept_count + (size_t)bh * Nb, i, Nb);
      w = wave_sum_i32(w);
      if (lane == 0) {
        plan[kPlanHdr + BH + bh] = w;
        w_head[bh] = w;
      }
    }
    __syncthreads();
    // rank by (work descending, index ascending)
    for (int bh = t; bh < BH; bh += kThreads) {
      const int w = w_head[bh];
      int r = 0;
      for (int j = 0; j < BH; ++j) {
        const int wj = w_head[j];
        r += (wj > w) || (wj == w && j < bh);
      }
      sorted[r] = bh;
    }
    __syncthreads();
    if (t < 64) {
      // greedy on one wavefront: lane x < 8 holds the load of XCD x (scaled to 32 bits;
      // +Nb per head: a row costs about one key block of fixed work); the minimum is a
      // register-only wave reduction, so a step costs no LDS round trips
      int shift = 0;
      while ((((long long)BH * Nb * (Nb + 1)) >> shift) > 0x3fffffffLL) ++shift;
      uint32_t load = t < kNumXcd ? 0u : 0xffffffffu;
      int nh = 0;
      for (int r = 0; r < BH; ++r) {
        const int bh = sorted[r];
        const uint32_t m = wave_min_u32(load);
        const unsigned long long is_min = __ballot(load == m);
        const int best = __ffsll((long long)is_min) - 1;  // least loaded XCD, lowest id on ties
        if (t == best) {
          xcd_of[bh] = best;
          rank_of[bh] = nh++;
          load += (uint32_t)(((long long)w_head[bh] + Nb) >> shift);
        }
      }
      if (t < kNumXcd) n_heads[t] = nh;
    }
  } else {
    if (t < kNumXcd) n_heads[t] = BH / kNumXcd + (t < BH % kNumXcd ? 1 : 0);
  }
  __syncthreads();
  if (t == 0) {
    int run = 0;
    for (int x = 0; x < kNumXcd; ++x) {
      off[x] = run;
      run += n_heads[x];
    }
  }
  __syncthreads();
  if (t < kNumXcd) {
    long long kept = 0;
    if (n_few < n_wg)  // (at most kFewHeads heads)
      for (int bh = 0; bh < BH; ++bh) kept += w_head[bh];
    const int first = list_first(working_groups(n_wg, n_few, kept, BH, Nb), t, BH);
    if (spread) spread[t * kCursorSpread] = first;
    plan[t] = spread ? n_heads[t] * Nb : first;
    plan[kNumXcd + t] = n_heads[t] * Nb;
    plan[2 * kNumXcd + t] = off[t];
  }
  for (int bh = t; bh < BH; bh += kThreads) {
    const int x = BH <= kPlanMaxHeads ? xcd_of[bh] : bh % kNumXcd;
    const int r = BH <= kPlanMaxHeads ? rank_of[bh] : bh / kNumXcd;
    plan[kPlanHdr + off[x] + r] = bh;
  }
}

// The Nb items of a head, longest kept list first, and, if `total` is given, the head's total kept
// count.  Stable counting sort by count class (class 0 = the longest rows).  Thread t < 256 owns a
// contiguous segment of the items and one column of the class histogram, so that items of a class
// keep their natural order.  The counts are first read once, coalesced and all in flight, and kept as
// class bytes in LDS when they fit (kStaged); otherwise the segments are read from global memory.
constexpr int kOrderStagedMax = 96 * 1024;  // items whose classes fit next to the histogram
template <bool kStaged, int kThreads>
__device__ __forceinline__ void class_order(const int *__restrict__ kept_count, int head, int Nb, uint32_t mult,
                                            int *__restrict__ seq, int *__restrict__ total, unsigned char *lds) {
  const int n = Nb;
  const int item0 = head * Nb;
  kept_count += item0;
  int *order = seq + item0;
  int(*hist)[kOrderCols] = reinterpret_cast<int(*)[kOrderCols]>(lds);
  int *scan = reinterpret_cast<int *>(lds) + kOrderClasses * kOrderCols;
  unsigned char *cls_lds = reinterpret_cast<unsigned char *>(scan + kOrderCols);  // [n] when kStaged
  const int t = threadIdx.x;
  const bool col = t < kOrderCols;
  const int per = (n + kOrderCols - 1) / kOrderCols;
  const int i0 = col ? min(n, t * per) : n, i1 = col ? min(n, i0 + per) : n;
  // class of a count c in [0, Nb]: (kOrderClasses-1) - floor(c * mult / 2^16) with
  // mult = floor((kOrderClasses-1) * 2^16 / Nb) from the host (no integer division here)
  auto cls = [&](int i) -> int {
    return (kOrderClasses - 1) - (int)(((uint32_t)row_count(kept_count, i, Nb) * mult) >> 16);
  };
  auto cls_of = [&](int i) -> int { return kStaged ? (int)cls_lds[i] : cls(i); };
  if (kStaged) {
#pragma unroll 4
    for (int i = t; i < n; i += kThreads) cls_lds[i] = (unsigned char)cls(i);
  }
  int *flat = &hist[0][0];
#pragma unroll 8
  for (int j = t; j < kOrderClasses * kOrderCols; j += kThreads) flat[j] = 0;
  __shared__ int sum_lds;
  if (t == 0) sum_lds = 0;
  __syncthreads();
  for (int i = i0; i < i1; ++i) hist[cls_of(i)][t] += 1;
  if (total) {
    int w = 0;
    for (int i = t; i < n; i += kThreads) w += row_count(kept_count, i, Nb);
    w = wave_sum_i32(w);
    if ((t & 63) == 0 && w) atomicAdd(&sum_lds, w);
  }
  __syncthreads();
  if (total && t == 0) total[head] = sum_lds;
  // exclusive scan over the histogram flattened class-major (index = class * 256 + column)
  int sum = 0;
  if (col)
    for (int j = 0; j < kOrderClasses; ++j) sum += flat[t * kOrderClasses + j];
  if (col) scan[t] = sum;
  __syncthreads();
  for (int d = 1; d < kOrderCols; d <<= 1) {
    const int add = col && t >= d ? scan[t - d] : 0;
    __syncthreads();
    if (col) scan[t] += add;
    __syncthreads();
  }
  if (col) {
    int run = scan[t] - sum;
    for (int j = 0; j < kOrderClasses; ++j) {
      const int x = flat[t * kOrderClasses + j];
      flat[t * kOrderClasses + j] = run;
      run += x;
    }
  }
  __syncthreads();
  for (int i = i0; i < i1; ++i) {
    const int b = cls_of(i);
    const int pos = hist[b][t];
    hist[b][t] = pos + 1;
    order[pos] = item0 + i;
  }
}

// The items of a head in batches of `batch` rows that walk through K/V together.  The rows an XCD
// works on at a time load more K/V blocks than its 4 MB L2 holds, so a block is found there only
// if other rows read it at about the same moment.  A batch is the longest row left and the rows
// whose lists are most like its list; inside a batch the longest row starts first.  Likeness: the
// list at eight evenly spaced ranks and its length, sum of absolute differences (as good as the
// overlap of the whole lists, which costs a pass over them).  Measured side by side with the other
// sequence, lists of the timed fields: L2 hits 57 -> 68 % at 40 heads, N = 32760, and 23 -> 45 % at 24 heads,
// N = 119056; attention with its plan 4617 -> 4510 us and 30.4 -> 29.3 ms, 16.2 -> 15.6 ms at 40 heads, N = 75600, 1376 ->
// 1365 us at 12 heads; no change for dense lists.
// One lane per row sorts the rows by length and gathers the samples; then one wavefront holds all
// rows in registers, sorted (RPL per lane, row 64 c + lane of the sorted order), and picks one
// batch after the other.
constexpr int kNearSamples = 8;
constexpr int kNearWords = kNearSamples / 2 + 1;  // pairs of 16-bit samples, and the length
template <int RPL>
__device__ __forceinline__ void near_order(const int *__restrict__ kept_idx, const int *__restrict__ kept_count,
                                           int head, int Nb, int batch, int *__restrict__ near_seq,
                                           unsigned char *lds) {
  uint32_t(*sig)[kNearMaxRows] = reinterpret_cast<uint32_t(*)[kNearMaxRows]>(lds);  // [kNearWords][rank]
  uint32_t *row_key = reinterpret_cast<uint32_t *>(sig + kNearWords);               // [rank]
  const int item0 = head * Nb;
  const int t = threadIdx.x, lane = t & 63;
  // bitonic sort, descending, of (length, lower index first), one key per lane (0 past the end)
  int P = 64;
  while (P < Nb) P <<= 1;
  uint32_t key = 0;
  if (t < Nb) key = ((uint32_t)row_count(kept_count + item0, t, Nb) << 10) | (uint32_t)(kNearMaxRows - 1 - t);
  for (int k = 2; k <= P; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      uint32_t other;
      if (j >= 64) {
        row_key[t] = key;
        __syncthreads();
        other = row_key[t ^ j];
        __syncthreads();
      } else {
        other = (uint32_t)__shfl_xor((int)key, j, 64);
      }
      const bool want_max = ((t & k) == 0) == ((t & j) == 0);
      key = want_max == (other > key) ? other : key;
    }
  if (t < Nb) {
    const int cnt = (int)(key >> 10), i = kNearMaxRows - 1 - (int)(key & (kNearMaxRows - 1));
    const int *list = kept_idx + (size_t)(item0 + i) * Nb;
    uint32_t s[kNearSamples];
#pragma unroll
    for (int k = 0; k < kNearSamples; ++k)
      s[k] = cnt > 0 ? (uint32_t)min(max(list[(cnt * (2 * k + 1)) / (2 * kNearSamples)], 0), Nb - 1) : 0u;
#pragma unroll
    for (int k = 0; k < kNearSamples / 2; ++k) sig[k][t] = s[2 * k] | (s[2 * k + 1] << 16);
    sig[kNearWords - 1][t] = (uint32_t)cnt * 4u;  // (a length counts like half of the samples)
    row_key[t] = (uint32_t)i;
  }
  __syncthreads();
  if (t >= 64) return;
  uint32_t w[RPL][kNearWords];
  int row[RPL];
  uint32_t left = 0;  // bit c: row 64 c + lane is not in the sequence yet
#pragma unroll
  for (int c = 0; c < RPL; ++c) {
    const int r = lane + 64 * c;
    if (r < Nb) left |= 1u << c;
    row[c] = (int)row_key[min(r, Nb - 1)];
#pragma unroll
    for (int k = 0; k < kNearWords; ++k) w[c][k] = sig[k][min(r, Nb - 1)];
  }
  const unsigned long long below_me = (1ull << lane) - 1ull;
  for (int done = 0; done < Nb;) {
    const int n = min(batch, Nb - done);
    int seed = -1;  // the longest row left
#pragma unroll
    for (int c = 0; c < RPL; ++c) {
      const unsigned long long b = __ballot((left >> c) & 1);
      if (seed < 0 && b) seed = 64 * c + __ffsll((long long)b) - 1;
    }
    uint32_t dist[RPL];
#pragma unroll
    for (int c = 0; c < RPL; ++c) dist[c] = 0;
#pragma unroll
    for (int k = 0; k < kNearWords; ++k) {
      const uint32_t ref = sig[k][seed];
#pragma unroll
      for (int c = 0; c < RPL; ++c) dist[c] = __builtin_amdgcn_sad_u16(w[c][k], ref, dist[c]);
    }
#pragma unroll
    for (int c = 0; c < RPL; ++c) dist[c] = (left >> c) & 1 ? dist[c] : 0xffffffffu;
    // the n-th smallest distance, bit by bit (all are below 12 * 1024 < 2^14)
    uint32_t v = 0;
    int n_less = 0;  // distances below v
    for (int bit = 13; bit >= 0; --bit) {
      const uint32_t cand = v | (1u << bit);
      int below = 0;
#pragma unroll
      for (int c = 0; c < RPL; ++c) below += __popcll(__ballot(dist[c] < cand));
      if (below < n) v = cand, n_less = below;
    }
    // every row below it and the first ones at it, in sorted order
    int eq_run = 0;
#pragma unroll
    for (int c = 0; c < RPL; ++c) {
      const bool eq = dist[c] == v;
      const unsigned long long e = __ballot(eq);
      const bool in = dist[c] < v || (eq && eq_run + __popcll(e & below_me) < n - n_less);
      eq_run += __popcll(e);
      const unsigned long long b = __ballot(in);
      if (in) {
        near_seq[item0 + done + __popcll(b & below_me)] = item0 + row[c];
        left &= ~(1u << c);
      }
      done += __popcll(b);
    }
  }
}

template <bool kStaged, int kThreads>
__global__ __launch_bounds__(kThreads) void attn_plan_kernel(const int *__restrict__ kept_idx,
                                                             const int *__restrict__ kept_count, int BH,
                                                             int Nb, int n_wg, int n_few, uint32_t mult, int batch,
                                                             const int *__restrict__ skip, int *__restrict__ plan,
                                                             int *__restrict__ spread, int *__restrict__ near_seq) {
  extern __shared__ __align__(16) unsigned char lds[];
  int id = blockIdx.x;
  if (skip && *skip == 0) {
    if (id == 0) {
      for (int i = threadIdx.x; i < BH; i += kThreads) plan[kPlanHdr + BH + i] = 0;
      if (threadIdx.x < kPlanHdr) plan[threadIdx.x] = 0;
      if (spread && threadIdx.x < kNumXcd) spread[threadIdx.x * kCursorSpread] = 0;
    }
    return;
  }
  if (kThreads == kPlanThreads && near_seq) {
    if (id < BH) {
      if (Nb <= 256)
        near_order<4>(kept_idx, kept_count, id, Nb, batch, near_seq, lds);
      else if (Nb <= 640)
        near_order<10>(kept_idx, kept_count, id, Nb, batch, near_seq, lds);
      else
        near_order<16>(kept_idx, kept_count, id, Nb, batch, near_seq, lds);
      return;
    }
    id -= BH;
  }
  if (id == 0) {
    plan_heads<kThreads>(kept_count, BH, Nb, n_wg, n_few, plan, spread, lds);
    return;
  }
  for (long long head = id - 1; head < BH; head += kPlanMaxGroups) {
    class_order<kStaged, kThreads>(kept_count, (int)head, Nb, mult, plan + kPlanHdr + 2 * BH,
                                   BH > kPlanMaxHeads ? plan + kPlanHdr + BH : nullptr, lds);
    __syncthreads();  // the LDS is free for the next head
  }
}

}  // namespace

int launch_attn_plan(int BH, int Nb, int n_wg, int n_few, int n_items, const int *kept_idx, const int *kept_count,
                     const int *skip, int *plan, size_t plan_bytes, const int **seq, int **cursors, hipStream_t st) {
  int *class_seq = plan + kPlanHdr + 2 * BH;
  int *near_seq = nullptr;
  // (with one row per workgroup there is nothing to order)
  const size_t near_bytes = attn_near_bytes(BH, Nb);
  if (near_bytes && BH <= kPlanMaxGroups && n_few == n_wg && n_items > n_wg && plan_bytes >= attn_plan_bytes(BH, Nb) + near_bytes)
    near_seq = class_seq + (size_t)BH * Nb;
  *seq = near_seq ? near_seq : class_seq;
  int *spread = nullptr;
  const size_t used = attn_plan_bytes(BH, Nb) + near_bytes;
  if (n_items > n_few && plan_bytes >= used + kCursorBytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(plan) + used;
    spread = reinterpret_cast<int *>((a + kCursorLine - 1) / kCursorLine * kCursorLine);
  }
  *cursors = spread;
  // rows an XCD works on at a time; twice as many with up to two heads per XCD on average, whose lists mostly
  // are walked in turn (kHeadsInTurn), so that their long rows start early (12 heads, N = 32760: 1407 -> 1359 us)
  int batch = (n_wg + kNumXcd - 1) / kNumXcd;
  if (BH <= 2 * kNumXcd) batch *= 2;
  const bool staged = Nb <= kOrderStagedMax;
  // with heads that are not ranked and short rows (no near_order) more workgroups per CU count for more than
  // lanes per head: 1048576 heads of one row 16.4 -> 9.8 ms
  const bool small = BH > kPlanMaxHeads && !near_seq;
  auto kern = small ? (staged ? attn_plan_kernel<true, kOrderCols> : attn_plan_kernel<false, kOrderCols>)
                    : (staged ? attn_plan_kernel<true, kPlanThreads> : attn_plan_kernel<false, kPlanThreads>);
  const size_t lds_class = (size_t)(kOrderClasses + 1) * kOrderCols * sizeof(int) + (staged ? (size_t)(Nb + 15) / 16 * 16 : 0);
  const size_t lds_other = (kNearWords + 1) * (size_t)kNearMaxRows * sizeof(int);  // >= plan_heads'
  static_assert(kNearWords >= 4 && kNearMaxRows >= kPlanMaxHeads, "LDS of plan_heads");
  const size_t lds = lds_class > lds_other ? lds_class : lds_other;
  if (lds > 64 * 1024) {
    const int dev = current_device();
    if (dev < 0) return fail(HEART_EHIP, "heart_block_sparse_attn: cannot identify the current device");
    static DeviceFlags attr_set[2];  // (only the staged kernels ask for more than 64 KB)
    const int most = (kOrderClasses + 1) * kOrderCols * (int)sizeof(int) + kOrderStagedMax;
    if (hipError_t e = set_max_lds_once(attr_set[small], dev, reinterpret_cast<const void *>(kern), most))
      return fail(HEART_EHIP, "hipFuncSetAttribute(plan kernel LDS): %s", hipGetErrorString(e));
  }
  const uint32_t mult = (uint32_t)(((kOrderClasses - 1) << 16) / Nb);
  const unsigned grid = (unsigned)(1 + (BH < kPlanMaxGroups ? BH : kPlanMaxGroups) + (near_seq ? BH : 0));
  hipLaunchKernelGGL(kern, dim3(grid), dim3(small ? kOrderCols : kPlanThreads), lds, st, kept_idx, kept_count, BH,
                     Nb, n_wg, n_few, mult, batch, skip, plan, spread, near_seq);
  return check_launch("attn_plan_kernel");
}

}  // namespace heart
