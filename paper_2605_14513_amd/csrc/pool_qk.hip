// heart_pool_qk: block means and token means of bf16 Q and K in one streaming pass
// (Alg. 1 step 1 and Eq. 4 for the token means; the block means feed the
// block-level importance ranking).  heart_pool_drift: the same pass, with the token means,
// the drift, the reuse rule and the layer gate (Eq. 4; Sec. 4.2; Alg. 1) together in ONE
// second launch instead of two (with few blocks, in the same one) -- the paper notes that fixed per-layer cost such as kernel
// launches caps what mask reuse can gain (Sec. 4.2, last paragraph).
//
// Bound by HBM reads: 2*B*H*N*D*2 bytes in, 2*B*H*(Nb+1)*D*4 bytes out.
//
// pool_blocks_kernel: one workgroup of 256 lanes per (tensor, b, h, block).
//   Every lane issues all of its 16-byte loads (8 bf16 each) before it uses any, so
//   a workgroup has its whole 32 KB block in flight; D/8 adjacent lanes cover one
//   token row, i.e. a wavefront reads whole contiguous rows.  Each lane sums its
//   rows in fp32 in row order, the 256/(D/8) row groups are combined through LDS
//   in a fixed order (no atomics on data: results are reproducible), and the block mean
//   is written once.
// Token means (token_mean_workgroup): one workgroup of 1024 lanes per (tensor, b, h) sums
//   block_mean * n_block over the blocks in fp64 in a fixed order and divides by N
//   (the mean of block means would be wrong when the last block is short).
//   heart_pool_qk runs it as a second small kernel (pool_token_mean_kernel).
// token_mean_drift_kernel (heart_pool_drift): the same token-mean workgroups; the one that
//   finishes the last token mean of a batch item -- found with a ticket counter in a caller
//   workspace that is zero on entry and zero again on return -- runs the drift stage for it
//   (drift_workgroup, the code of heart_drift).  No workgroup waits for another.
//   The eight XCDs of the chip have separate L2 caches and a device-wide fence writes back and
//   invalidates a whole L2, so the values that cross workgroups (the token means) move with
//   device-scope atomic stores and loads instead; a workgroup waits for the acknowledgement of
//   its stores before it takes its ticket.
//   The anchors are written from the registers that were compared instead of after a second pass of
//   loads (D = 128; 10.2 -> 9.3 us at 40 heads of 256 blocks).
// pool_drift_small_kernel (heart_pool_drift of few blocks): everything in one launch.
//   (Doing the same in the tail of pool_blocks_kernel at full size, one ticket per block, was measured: a
//   device-wide fence per workgroup took the launch from 0.12 to 3.4 ms, device-scope stores
//   with a ticket per workgroup to 0.23 ms -- under 6 TB/s of reads the store acknowledgement
//   and the atomic's round trip double the lifetime of a workgroup -- so the pooling pass
//   itself stays free of cross-workgroup traffic.)
#include "drift_device.h"
#include "heart_internal.h"

namespace heart {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kPoolThreads = 256;       // pooling pass: lanes per workgroup
constexpr int kMeanThreads = 1024;      // token means (and the drift stage behind them): lanes per workgroup
constexpr int kTokenMeanBatch = 8;      // block means in flight per lane
constexpr int kMeanLdsDoubles = kMeanThreads * 4;  // 32 KB: token-mean slices (fp64); reused for the drift marks

// Device-scope (all XCDs) store of a value that another workgroup of the same launch will read
// (with a device-scope load): coherent across the L2 caches of the XCDs without a cache-wide
// fence.
__device__ __forceinline__ void store_device_scope(float *p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// This wavefront's global stores have been acknowledged (for device-scope stores: at the level
// every XCD sees).
__device__ __forceinline__ void wait_for_own_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Token mean of one (tensor, b, h): src = its block means [Nb][D], dst = [D].  Lanes are
// arranged as D/4 column groups (float4 each) times 1024/(D/4) block slices; each slice adds
// its blocks in increasing block order in fp64, slices are combined in slice order.  Called
// by a whole workgroup of kMeanThreads lanes (contains a barrier); part: LDS, kMeanLdsDoubles
// doubles.
// kAcross: dst is read by another workgroup of this launch (device-scope stores); the
// arithmetic is the same either way.
template <int D, bool kAcross>
__device__ __forceinline__ void token_mean_workgroup(const float *src, int N, int block, int Nb,
                                                     float *dst, double *part) {
  constexpr int CG = D / 4;             // column groups
  constexpr int SL = kMeanThreads / CG; // slices over the blocks
  static_assert(SL * D <= kMeanLdsDoubles, "LDS of the token mean");
  const int cg = threadIdx.x % CG, sl = threadIdx.x / CG;
  const int per = (Nb + SL - 1) / SL;
  const int i0 = sl * per, i1 = min(Nb, i0 + per);
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  // (the loads of kTokenMeanBatch blocks are issued before any is used: the kernel is bound by
  // memory round trips; the order of the additions is the block order either way)
  for (int ib = i0; ib < i1; ib += kTokenMeanBatch) {
    float4 m[kTokenMeanBatch];
#pragma unroll
    for (int u = 0; u < kTokenMeanBatch; ++u) {
      const int i = min(ib + u, i1 - 1);
      m[u] = *reinterpret_cast<const float4 *>(src + (size_t)i * D + cg * 4);
    }
#pragma unroll
    for (int u = 0; u < kTokenMeanBatch; ++u) {
      const int i = ib + u;
      if (i < i1) {
        const double n = (double)min(block, N - i * block);
        a0 += (double)m[u].x * n;
        a1 += (double)m[u].y * n;
        a2 += (double)m[u].z * n;
        a3 += (double)m[u].w * n;
      }
    }
  }
  part[sl * D + cg * 4 + 0] = a0;
  part[sl * D + cg * 4 + 1] = a1;
  part[sl * D + cg * 4 + 2] = a2;
  part[sl * D + cg * 4 + 3] = a3;
  __syncthreads();
  if (threadIdx.x < D) {
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < SL; ++r) s += part[r * D + threadIdx.x];
    if constexpr (kAcross)
      store_device_scope(dst + threadIdx.x, (float)(s / (double)N));
    else
      dst[threadIdx.x] = (float)(s / (double)N);
  }
}

struct PoolDriftArgs {  // what the drift stage needs beyond the token-mean arguments
  float *qanchor, *kanchor;
  unsigned char *has_anchor;
  const float *delta;
  float gate_lo, gate_hi;
  int commit;
  float *drift;
  unsigned char *refresh;
  unsigned *tickets;  // [B]; zero on entry, zero on return
};

// Mean of one block, by kPoolThreads lanes (`t` = 0 .. kPoolThreads - 1) that all call it, of a head's rows n0 ..
// n0 + nrows - 1 (at `base`, token stride sn); contains a barrier of the workgroup.  part: LDS, kPoolPart floats.
// kThrough: the mean goes out with device-scope stores (dst is read by another workgroup of this launch, or see
// pool_blocks_kernel).  nrows <= 0: no block for these lanes.  also(): called once the loads are on their way.
constexpr int kPoolPart = kPoolThreads * 8;
template <int D, bool kThrough, class Also>
__device__ __forceinline__ void block_mean(const uint16_t *base, int n0, long long sn, int nrows, float *dst, float *part, int t,
                                           Also also) {
  constexpr int LPR = D / 8;               // lanes per token row
  constexpr int RPP = kPoolThreads / LPR;  // rows per pass
  constexpr int MAXP = 128 / RPP;          // passes for the largest block (128 tokens)
  static_assert(RPP * D == kPoolPart, "LDS of the block mean");
  const int lane_col = (t % LPR) * 8;
  const int row0 = t / LPR;

  uint4 v[MAXP];
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    int r = row0 + p * RPP;
    v[p] = make_uint4(0u, 0u, 0u, 0u);
    if (r < nrows) {
      // streaming read: every byte is used once by this kernel
      const u32x4 x = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(base + (long long)(n0 + r) * sn + lane_col));
      v[p] = make_uint4(x.x, x.y, x.z, x.w);
    }
  }
  also();
  float acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = 0.f;
#pragma unroll
  for (int p = 0; p < MAXP; ++p) {
    acc[0] += bf16lo(v[p].x);
    acc[1] += bf16hi(v[p].x);
    acc[2] += bf16lo(v[p].y);
    acc[3] += bf16hi(v[p].y);
    acc[4] += bf16lo(v[p].z);
    acc[5] += bf16hi(v[p].z);
    acc[6] += bf16lo(v[p].w);
    acc[7] += bf16hi(v[p].w);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[row0 * D + lane_col + e] = acc[e];
  __syncthreads();
  if (t < D && nrows > 0) {
    float s = 0.f;
#pragma unroll
    for (int r = 0; r < RPP; ++r) s += part[r * D + t];
    if constexpr (kThrough)
      store_device_scope(dst + t, s / (float)nrows);
    else
      dst[t] = s / (float)nrows;
  }
}

// kStream: a call whose Q and K do not stay in the chip's memory-side cache.  Read from HBM without the stores of the
// block means, the pass ran 10 to 13 % faster although they are 1.5 % of the bytes: a plain store leaves a dirty line in
// the L2 of an XCD, to be written back whenever the reads of the stream push it out.  There the means are therefore written
// through (device scope), and 2^run consecutive blocks (128 KB of rows, and their means) go to one XCD.
// (workgroup w is taken to run on XCD w % 8; what it computes does not depend on it.)
template <int D, bool kStream>
__global__ __launch_bounds__(kPoolThreads) void pool_blocks_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, long long qsb, long long qsh,
    long long qsn, long long ksb, long long ksh, long long ksn, int H, int N, int block, int Nb,
    int run, float *__restrict__ qblk, float *__restrict__ kblk) {
  __shared__ float part[kPoolPart];

  unsigned w = blockIdx.x;
  if constexpr (kStream) {
    const unsigned at = w >> (run + 3);                                       // which 8 * 2^run workgroups
    if ((at + 1) << (run + 3) <= gridDim.x)                                   // (the last ones, if fewer, stay in order)
      w = (((at << 3) + (w & 7u)) << run) + ((w >> 3) & ((1u << run) - 1u));
  }
  // w enumerates (b*H+h, tensor, block) with the block index fastest so
  // that consecutive workgroups stream consecutive memory.  (Divisions in 32 bits, which hold the
  // grid: 13.85 -> 13.4 us for heart_pool_drift of two items of 10 heads of 101 blocks of 64.)
  const unsigned rest = w / (unsigned)Nb;  // = 2 * (b*H+h) + tensor
  const int i = (int)(w - rest * (unsigned)Nb), which = (int)(rest & 1u);
  const unsigned bh = rest >> 1;
  const int b = (int)(bh / (unsigned)H), h = (int)(bh - (unsigned)b * (unsigned)H);

  const uint16_t *base = which ? (k + b * ksb + h * ksh) : (q + b * qsb + h * qsh);
  long long sn = which ? ksn : qsn;
  const int n0 = i * block;
  block_mean<D, kStream>(base, n0, sn, min(block, N - n0),
                       (which ? kblk : qblk) + ((size_t)bh * Nb + i) * D, part, (int)threadIdx.x, [] {});
}

// One workgroup per (tensor, b, h).
template <int D>
__global__ __launch_bounds__(kMeanThreads) void pool_token_mean_kernel(const float *__restrict__ qblk,
                                                                       const float *__restrict__ kblk,
                                                                       int N, int block, int Nb,
                                                                       float *__restrict__ qmean,
                                                                       float *__restrict__ kmean) {
  __shared__ double part[kMeanLdsDoubles];
  const int which = blockIdx.x & 1;
  const long long bh = blockIdx.x >> 1;
  token_mean_workgroup<D, false>((which ? kblk : qblk) + (size_t)bh * Nb * D, N, block, Nb,
                                 (which ? kmean : qmean) + (size_t)bh * D, part);
}

// The same, and the workgroup that completes a batch item runs the drift stage.  A ticket
// (device-scope atomic) is taken after this workgroup's device-scope stores have been
// acknowledged (wait, then barrier, then the atomic of one lane); the workgroup that draws the
// last ticket of its batch item then reads every token mean with device-scope loads.
template <int D>
__global__ __launch_bounds__(kMeanThreads) void token_mean_drift_kernel(
    const float *__restrict__ qblk, const float *__restrict__ kblk, int H, int N, int block, int Nb,
    float *qmean, float *kmean, PoolDriftArgs fa) {
  __shared__ double lds[kMeanLdsDoubles];
  __shared__ int s_last;
  const int which = blockIdx.x & 1;
  const long long bh = blockIdx.x >> 1;
  const int b = (int)(bh / H);
  token_mean_workgroup<D, true>((which ? kblk : qblk) + (size_t)bh * Nb * D, N, block, Nb,
                                (which ? kmean : qmean) + (size_t)bh * D, lds);
  wait_for_own_stores();
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned t = atomicAdd(&fa.tickets[b], 1u);
    s_last = (t == 2u * (unsigned)H - 1u);
    if (s_last) atomicExch(&fa.tickets[b], 0u);  // nobody else touches it any more in this launch
  }
  __syncthreads();
  if (!s_last) return;
  // (asked for before the block means, by every workgroup: 13.6 -> 14.1 us for a call of two items of 10 heads of 101 blocks.  At D =
  // 64 they are loaded with the means: ahead of them 72 heads of one block took 11.3 instead of 10.9 us, 200 of ten 22.5
  // instead of 21.6; at D = 128 it is the other way round, 12.6 against 13.1 and 38.8 against 39.6)
  DriftAnchors<D / 64> anchors;
  if constexpr (D == 128)
    anchors.load(b, (int)(threadIdx.x >> 6) * kDriftHeadsPerPass, H, D, fa.qanchor, fa.kanchor, fa.has_anchor, fa.delta);
  const size_t item = (size_t)b * H * D;
  // (at D = 64 few lanes would write the kept means: 13.7 -> 13.85 us for that call)
  drift_workgroup<D / 64, D == 128, D == 128>(b, H, D, DriftMeansAcross{qmean + item, kmean + item}, anchors, fa.qanchor,
                                              fa.kanchor, fa.has_anchor, fa.delta, fa.gate_lo, fa.gate_hi, fa.commit,
                                              fa.drift, fa.refresh, reinterpret_cast<unsigned char *>(lds));
}

// All of heart_pool_drift in one launch, for few blocks, where it is bound by launches and by a chain of memory round
// trips (block, acknowledgement, ticket, block means, result; 7.1 us at two heads of 16 blocks of 64, D = 64): a workgroup
// pools kSmallBlocks blocks of a batch item, the last one of the item computes its token means (in block order in fp64 as
// token_mean_workgroup does, which has at most one block a slice here, so the bits are the same), keeps them in LDS and runs
// the drift stage.
constexpr int kSmallBlocks = kMeanThreads / kPoolThreads;
constexpr int kSmallMeans = kSmallBlocks * kPoolPart;  // token means that fit
constexpr int kSmallMarks = 2 * 32;                   // two bytes a head, 32 heads
template <int D>
__global__ __launch_bounds__(kMeanThreads) void pool_drift_small_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, long long qsb, long long qsh, long long qsn,
    long long ksb, long long ksh, long long ksn, int H, int N, int block, int Nb, int per_item, float *qblk, float *kblk,
    float *__restrict__ qmean, float *__restrict__ kmean, PoolDriftArgs fa) {
  __shared__ float lds[kSmallMeans];
  __shared__ unsigned char marks[kSmallMarks];
  __shared__ int s_last;
  const int b = (int)(blockIdx.x / per_item), group = threadIdx.x / kPoolThreads;
  DriftAnchors<D / 64> anchors;  // (any workgroup may become the one that needs them)
  {
    const int p = (int)(blockIdx.x % per_item) * kSmallBlocks + group;  // (h, tensor, block)
    const int i = p % Nb, which = (p / Nb) & 1, h = p / Nb >> 1, n0 = i * block;
    const long long sn = which ? ksn : qsn;
    const uint16_t *base = which ? (k + b * ksb + h * ksh) : (q + b * qsb + h * qsh);
    block_mean<D, true>(base, n0, sn, h < H ? min(block, N - n0) : 0,
                        (which ? kblk : qblk) + (((size_t)b * H + h) * Nb + i) * D, lds + group * kPoolPart,
                        (int)(threadIdx.x % kPoolThreads), [&]() __attribute__((always_inline)) {
                          anchors.load(b, (int)(threadIdx.x >> 6) * kDriftHeadsPerPass, H, D, fa.qanchor, fa.kanchor,
                                       fa.has_anchor, fa.delta);
                        });
  }
  wait_for_own_stores();
  __syncthreads();
  if (threadIdx.x == 0) {
    const unsigned t = atomicAdd(&fa.tickets[b], 1u);
    s_last = t == (unsigned)per_item - 1u;
    if (s_last) atomicExch(&fa.tickets[b], 0u);
  }
  __syncthreads();
  if (!s_last) return;
  const size_t item = (size_t)b * H * D;
  const int n = H * D;
  for (int c = threadIdx.x; c < 2 * n; c += kMeanThreads) {
    const int which = c >= n, o = c - which * n;
    const float *src = (which ? kblk : qblk) + (item + (size_t)(o / D) * D) * Nb + o % D;
    double s = 0.0;
    for (int ib = 0; ib < Nb; ib += kTokenMeanBatch) {
      float m[kTokenMeanBatch];
#pragma unroll
      for (int u = 0; u < kTokenMeanBatch; ++u)
        m[u] = __hip_atomic_load(src + (size_t)min(ib + u, Nb - 1) * D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
      for (int u = 0; u < kTokenMeanBatch; ++u)
        if (ib + u < Nb) s += (double)m[u] * (double)min(block, N - (ib + u) * block);
    }
    const float mean = (float)(s / (double)N);
    lds[c] = mean;
    (which ? kmean : qmean)[item + o] = mean;
  }
  __syncthreads();
  drift_workgroup<D / 64, true, true>(b, H, D, DriftMeans{lds, lds + n}, anchors, fa.qanchor, fa.kanchor, fa.has_anchor,
                                      fa.delta, fa.gate_lo, fa.gate_hi, fa.commit, fa.drift, fa.refresh, marks);
}

// Largest calls of pool_drift_small_kernel: workgroups of a batch item and in all (one ticket each, served one after another),
// token means of a batch item (one workgroup makes them all, a lane one or two of them) and blocks a head (a chain of loads).
// heart_pool_drift in two launches -> in one, us: D = 64, H x Nb = 2 x 16 7.9 -> 7.1, 8 x 8 (32 workgroups) 8.1 -> 7.2, 16 x
// 4 (32 workgroups, 2048 means) 8.5 -> 8.1, 10 x 8 (40) 8.0 -> 7.6, 2 x 24 8.1 -> 7.4, six heads of 8 in 8 items (192 workgroups)
// 9.5 -> 9.0; beyond: 10 x 9 (45) 8.1 -> 8.5, 25 x 1 (3200) 8.2 -> 8.7, 2 x 40 8.0 -> 8.4, 8 items of 32 9.5 -> 10.1.  D = 128,
// where the two launches keep the means they compared: 2 x 16 8.2 -> 7.8, 4 x 8 (16 workgroups, 1024 means) 8.6 -> 7.9, 3 x
// 10 8.2 -> 8.1; beyond: 2 x 24 (24) 8.6 -> 8.8, 8 x 1 (2048 means) 7.8 -> 8.4, 25 x 3 8.8 -> 13.3.
constexpr int kSmallLaunch = 192, kSmallNb = 24;
template <int D>
constexpr int kSmallItem = D == 64 ? 40 : 16;
template <int D>
constexpr int kSmallCols = D == 64 ? 2048 : 1024;
static_assert(kSmallNb <= kMeanThreads / (128 / 4), "at most one block a slice of the token means");
static_assert(kSmallCols<64> <= kSmallMeans && kSmallCols<64> / 64 <= kSmallMarks, "LDS");
// Whether pool_blocks_kernel<D, true> is the better one: where Q and K are more bytes than the 256 MiB of the memory-side cache, and
// one and a half times as many with blocks of 32 KB, which write half as many means.  heart_pool_qk with plain stores in block order ->
// written through in runs, us: D = 128, blocks of 128, H x N = 40 x 32760 113.5 -> 107.8, 24 x 119056 250 -> 234.5 (5.8 -> 6.2 TB/s),
// 24 x 32760 (383 MiB) 73.7 -> 72.0, but three items of 40 x 5000 (292) 60.1 -> 60.4, five of 8 x 16000 (312) 57.0 -> 57.5; blocks of 64
// 40 x 32760 116.5 -> 110.2, 22 items of 8 x 3000 (257) 59.5 -> 57.2; D = 64, 80 x 32760 113.3 -> 104.4, 48 x 119056 244 -> 227.7, 99
// items of 12 x 1000 (290) 60.3 -> 58.6; below the cache's size 13 x 32760 38.3 -> 39.1, 28 x 32760 of D = 64 40.1 -> 40.6 and a call of
// 10 heads of 101 blocks 0.5 us more (there the token means find the plain stores in an L2).  Written through in block order 110.4 and
// 236.4; plain stores with a contiguous eighth of the blocks on each XCD 110.5 and 244.
// Runs of 64, 128, 256 KB: 110.4, 107.3, 109.4 and 242.5, 235.4, 235.8.
// Rows between those of other heads: of D = 64 nothing is gained (82.6 -> 83.1, four items of 24 heads of 20000 tokens).  Of D = 128 long
// heads gain from 480 MiB on (40 x 32760 116.6 -> 114.0, two items of 24 x 32760 140.8 -> 134.5; 17 x 32760 50.5 -> 51.7, two of 10 x 32760
// 58.1 -> 59.5, eight of 40 x 3000 (468 MiB) 95.6 -> 96.2), with blocks of 64 from 256 (12 of 8 x 8191 75.2 -> 70.0, three of 24 x 8191
// 57.3 -> 56.3).  Short heads lose more often than they gain: 105 items of 40 x 130 87.7 -> 93.5, 46 of 40 x 500 86.5 -> 91.8, 27 of 40 x
// 500 in blocks of 64 55.1 -> 57.2, 17 of 40 x 1000 62.2 -> 63.5, against 638 of 8 x 257 144.8 -> 138.8.
static bool pool_streams(const heart_shape &s) {
  const long long bytes = 4LL * s.B * s.H * s.N * s.D, MiB = 1LL << 20;
  const bool small = s.block * s.D <= 8192;
  if (s.q_stride[2] == s.D && s.k_stride[2] == s.D) return bytes > (small ? 256 : 384) * MiB;
  return s.D == 128 && s.N >= 2000 && bytes > (small ? 256 : 480) * MiB;
}
constexpr int kRunBytes = 128 * 1024;
template <int D>
static int launch_pool_t(const heart_shape &s, const uint16_t *qp, const uint16_t *kp, float *qblk,
                         float *kblk, float *qmean, float *kmean, const PoolDriftArgs *fused,
                         hipStream_t st) {
  const int Nb = (s.N + s.block - 1) / s.block;
  const long long nwg = 2LL * s.B * s.H * Nb;
  if (nwg > 0x7fffffffLL) return fail(HEART_EUNSUPPORTED, "heart_pool_qk: grid too large");
  const long long per_item = (2LL * s.H * Nb + kSmallBlocks - 1) / kSmallBlocks;
  if (fused && Nb <= kSmallNb && 2 * s.H * D <= kSmallCols<D> && per_item <= kSmallItem<D> && s.B * per_item <= kSmallLaunch) {
    hipLaunchKernelGGL(pool_drift_small_kernel<D>, dim3((unsigned)(s.B * per_item)), dim3(kMeanThreads), 0, st, qp, kp,
                       s.q_stride[0], s.q_stride[1], s.q_stride[2], s.k_stride[0], s.k_stride[1], s.k_stride[2], s.H, s.N,
                       s.block, Nb, (int)per_item, qblk, kblk, qmean, kmean, *fused);
    return check_launch("pool_drift_small_kernel");
  }
  const dim3 grid((unsigned)nwg), blk(kPoolThreads), grid2((unsigned)(2 * s.B * s.H)), blk2(kMeanThreads);
  const bool stream = pool_streams(s);
  int run = 2;
  while ((s.block * D * 2) << run < kRunBytes) ++run;
  hipLaunchKernelGGL((stream ? pool_blocks_kernel<D, true> : pool_blocks_kernel<D, false>), grid, blk, 0, st, qp, kp,
                     s.q_stride[0], s.q_stride[1], s.q_stride[2], s.k_stride[0], s.k_stride[1], s.k_stride[2], s.H, s.N,
                     s.block, Nb, run, qblk, kblk);
  if (int rc = check_launch("pool_blocks_kernel")) return rc;
  if (fused) {
    hipLaunchKernelGGL(token_mean_drift_kernel<D>, grid2, blk2, 0, st, qblk, kblk, s.H, s.N, s.block,
                       Nb, qmean, kmean, *fused);
    return check_launch("token_mean_drift_kernel");
  }
  hipLaunchKernelGGL(pool_token_mean_kernel<D>, grid2, blk2, 0, st, qblk, kblk, s.N, s.block, Nb,
                     qmean, kmean);
  return check_launch("pool_token_mean_kernel");
}

int launch_pool(const heart_shape &s, const void *q, const void *k, float *qblk, float *kblk,
                float *qmean, float *kmean, hipStream_t st) {
  const uint16_t *qp = (const uint16_t *)q, *kp = (const uint16_t *)k;
  if (s.D == 128) return launch_pool_t<128>(s, qp, kp, qblk, kblk, qmean, kmean, nullptr, st);
  return launch_pool_t<64>(s, qp, kp, qblk, kblk, qmean, kmean, nullptr, st);
}

int launch_pool_drift(const heart_shape &s, const void *q, const void *k, float *qblk, float *kblk,
                      float *qmean, float *kmean, float *qanchor, float *kanchor,
                      unsigned char *has_anchor, const float *delta, float gate_lo, float gate_hi,
                      int commit, float *drift, unsigned char *refresh, unsigned *tickets,
                      hipStream_t st) {
  const uint16_t *qp = (const uint16_t *)q, *kp = (const uint16_t *)k;
  const PoolDriftArgs fa{qanchor, kanchor, has_anchor, delta, gate_lo, gate_hi,
                         commit, drift, refresh, tickets};
  if (s.D == 128) return launch_pool_t<128>(s, qp, kp, qblk, kblk, qmean, kmean, &fa, st);
  return launch_pool_t<64>(s, qp, kp, qblk, kblk, qmean, kmean, &fa, st);
}

}  // namespace heart
