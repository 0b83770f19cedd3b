// Error-guided Budgeted Calibration (Sec. 4.3): the two computations that turn measured
// velocities into per-head thresholds.
//
//  heart_ebc_band_error   the frequency-weighted velocity error of Eq. 6 on the GPU.
//    The four bands of the appendix (after fftshift a frequency is low along an axis of
//    length n when it lies within floor(n/4) of the centre) are products of per-axis
//    low / high sets, and the low set {-r..r}, r = floor(n/4), is symmetric: the low part of
//    a line is spanned by the 2r+1 real functions 1, cos(2 pi f j / n), sin(2 pi f j / n),
//    f = 1..r, which are orthogonal.  With c_k the sums of a line against them,
//        |P e|^2 = 1/n (c_0^2 + 2 sum_{k>0} c_k^2)
//    so, with S_A the weighted sum of squares after contracting the axes in A (weight 2 per
//    axis with k > 0, no rounding) and n_tot = T*Y*X, the unnormalised transform of the
//    definition gives by Parseval
//        n_tot |Pt e|^2 = Y X S_T    n_tot |Py Px e|^2 = T S_XY    n_tot |Pt Py Px e|^2 = S_XYT
//        E_LL = S_XYT                E_LH = Y X S_T - S_XYT
//        E_HL = T S_XY - S_XYT       E_HH = n_tot |e|^2 - Y X S_T - T S_XY + S_XYT
//    and the denominator is n_tot |dense|^2 + epsilon.  About n/2 coefficients of an axis are
//    all that is ever computed or stored of it: no transform, no projected tensor.
//    The contractions run on the fp64 matrix cores (v_mfma_f64_16x16x4_f64: 16 coefficients
//    of 16 lines, four elements of the lines a step); the sums of squares are taken from the
//    accumulators and reduced in a fixed order.  Two launches for latents:
//      ebc_first   x coefficients of err with |err|^2, S_T of err, |dense|^2
//      ebc_plane   y and t coefficients of the x coefficients with S_XY and S_XYT; its last workgroup adds everything up
//    or, where t is longer than 63 or y than 48, in the place of the second
//      ebc_second  y coefficients of the x coefficients with S_XY
//      ebc_third   S_XYT; its last workgroup adds everything up
//    Bound by latency: at 128 x 21 x 30 x 52 the matrix instructions are 7 us of the chip and the
//    90 MB moved (half of them in the caches) some 18 us; the launches take 20 + 13 us, of
//    which a table, a first load and a last sum each about 1 us.  Whole call 41.6 -> 33.0 us against three
//    launches that counted 400 workgroups on one ticket, 257 us with twelve launches that convolved in fp64 on the
//    vector units (results equal to 1e-15); 128 x 33 x 45 x 80 134 -> 119 us, 16 x 21 x 30 x 52 21.3 -> 16.7 us.
//    A calibration run evaluates this once per (head, candidate, prompt-step), off the serving path.
//
//  heart_ebc_select       the one-candidate-per-head selection of Eq. 5 (minimum summed
//    error under a mean-sparsity budget), solved exactly on the host: linear relaxation of
//    the multiple-choice knapsack (per-head lower convex hulls, increments in order of
//    error per unit of sparsity) as the bound of a depth-first branch and bound on the one
//    head the relaxation leaves fractional.  Replaces the generic integer-program solver
//    the paper uses.
#include <algorithm>
#include <cmath>
#include <vector>

#include "heart_internal.h"

namespace heart {

constexpr int kEbcThreads = 256;
constexpr int kEbcWaves = kEbcThreads / 64;
constexpr int kEbcMaxAxis = 1024;   // longest axis (the trigonometric table sits in LDS)
constexpr int kEbcPartials = 1024;  // partial sums per reduction, one per workgroup
constexpr int kEbcSums = 5;         // |e|^2, S_T, S_XY, S_XYT, |dense|^2
constexpr int kEbcTileCols = 32;    // lines a wavefront contracts at a time (two matrix tiles)
typedef __attribute__((ext_vector_type(4))) double ebc_f64x4;

__host__ __device__ constexpr int ebc_coefs(int n) { return 2 * (n / 4) + 1; }

// cos(2 pi m / n) in tab[m], sin(2 pi m / n) in tab[n + m], by the whole workgroup
__device__ __forceinline__ void ebc_table(int n, double *tab) {
  for (int m = threadIdx.x; m < n; m += kEbcThreads) {
    double c, s;
    sincospi(2.0 * (double)m / (double)n, &s, &c);
    tab[m] = c;
    tab[n + m] = s;
  }
  __syncthreads();
}

// sum over the workgroup in a fixed order, valid in thread 0; red: kEbcWaves doubles of LDS
__device__ __forceinline__ double ebc_block_sum(double v, double *red) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = red[0];
#pragma unroll
  for (int w = 1; w < kEbcWaves; ++w) s += red[w];
  return s;
}

// A tensor as lines of n elements: element j of line o * inner + s is in[(o * n + j) * inner + s].
// Coefficient k of line c goes to out[k * lines + c] (the store is then coalesced, and the next
// axis of the original tensor is the last one of the result).
// Weight of a line in the sum of squares: 1, or 2 per earlier axis with k > 0.  With c = c1 * wdiv
// + c0, c1 = ky * wmod + kx counts the coefficients of the earlier axes.
struct EbcLines {
  int n;
  long long inner, lines;
  long long wdiv;  // 0: all weights are 1
  int wmod;
  int share;  // wavefronts that the coefficients of 32 lines are dealt over, in pairs of 16
};

__device__ __forceinline__ long long ebc_div(long long a, long long b) {
  if (((unsigned long long)(a | b) >> 32) == 0) return (long long)((uint32_t)a / (uint32_t)b);
  return a / b;
}

// 32 lines as one wavefront contracts them: lane l16 = lane % 16 holds lines col0 + l16 and
// col0 + 16 + l16, lane group g = lane / 16 their elements j = g mod 4; of lines whose elements lie side by side (kUnit)
// instead elements 4 g .. 4 g + 3 of every whole 16, which are one load: the loads of single elements took four times
// the instructions, and 16 wavefronts more lines than the 32 KB cache has (128 x 33 x 45 x 80: 124 -> 119 us).
template <typename TIn>
struct EbcTile {
  long long col0;
  const TIn *src[2];  // the lines (kUnit), or this lane's first elements
  bool ok[2];         // the line exists (others count as zeros)
};
template <typename TIn, bool kUnit>
__device__ __forceinline__ EbcTile<TIn> ebc_tile_at(const TIn *in, const EbcLines &L, long long tile) {
  const int l16 = threadIdx.x & 15, g = (threadIdx.x & 63) >> 4;
  EbcTile<TIn> t;
  t.col0 = tile * kEbcTileCols;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const long long col = t.col0 + 16 * c + l16;
    t.ok[c] = col < L.lines;
    const long long o = kUnit ? col : ebc_div(col, L.inner);
    t.src[c] = in + (kUnit ? col * L.n : (o * L.n + g) * L.inner + (col - o * L.inner));
  }
  return t;
}

constexpr int kEbcBatch = 4;  // contraction steps (of 4 elements) whose loads are issued together
template <typename TIn>
struct EbcBatch {
  TIn v[kEbcBatch][2];
};
template <typename TIn>
struct __attribute__((packed, aligned(sizeof(TIn)))) EbcQuad {
  TIn v[kEbcBatch];
};
template <typename TIn, bool kUnit>
__device__ __forceinline__ void ebc_load(EbcBatch<TIn> &d, const EbcTile<TIn> &t, const EbcLines &L, int j0) {
  const int g = (int)((threadIdx.x & 63) >> 4);
  if (kUnit && j0 + 4 * kEbcBatch <= L.n) {  // uniform
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      EbcQuad<TIn> x{};
      if (t.ok[c]) x = *reinterpret_cast<const EbcQuad<TIn> *>(t.src[c] + j0 + 4 * g);
#pragma unroll
      for (int u = 0; u < kEbcBatch; ++u) d.v[u][c] = x.v[u];
    }
    return;
  }
  const long long inner = kUnit ? 1 : L.inner;
  const int last = L.n - g;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const TIn *p = t.src[c] + j0 * inner + (kUnit ? g : 0);
#pragma unroll
    for (int u = 0; u < kEbcBatch; ++u) d.v[u][c] = t.ok[c] && j0 + 4 * u < last ? p[4 * u * inner] : (TIn)0;
  }
}

// i, less n from n on
__device__ __forceinline__ int ebc_wrap(int i, int n) { return (int)min((uint32_t)i, (uint32_t)(i - n)); }

// M * 16 coefficients from kt * 16 on of a tile; `cur` holds its first batch, and that of `next` on return
template <int M, typename TIn, bool kUnit, bool kStore, bool kSumIn>
__device__ __forceinline__ void ebc_tile(EbcBatch<TIn> &cur, const EbcTile<TIn> &t, const EbcTile<TIn> &next,
                                         double *__restrict__ out, const EbcLines &L, const double *tab, int kt,
                                         int K, double &e_out, double &e_in) {
  // operand layout (16x16x4 fp64): A lane = (row lane%16, k lane/16), B lane = (k lane/16, column
  // lane%16), D lane register r = (row lane/16 + 4 r, column lane%16)
  const int lane = threadIdx.x & 63, l16 = lane & 15, g = lane >> 4;
  const int n = L.n;
  ebc_f64x4 acc[M][2];
  // (f * j) mod n at this lane's j, its step to the j of the next contraction step (j + 4, or of a whole 16 of a unit line
  // j + 1: f itself, which is at most n / 4), table half.  (The step from a whole 16 to the next is made from f each time: as
  // one more array it took 8 to 13 registers to scratch memory; 16 x 3 x 56 x 52 23.2 -> 21.8 us, 16 x 8 x 1024 x 8 101 -> 81.)
  int idx[M], step[M], part[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int k = (kt + m) * 16 + l16;
    const int f = k < K ? (k + 1) >> 1 : 0;  // (coefficients past K are computed and dropped)
    part[m] = (k & 1) == 0 && k > 0 && k < K ? n : 0;
    idx[m] = (int)((uint32_t)(f * (kUnit ? 4 * g : g)) % (uint32_t)n);
    step[m] = (int)((uint32_t)(kUnit ? f : 4 * f) % (uint32_t)n);
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[m][c] = ebc_f64x4{0.0, 0.0, 0.0, 0.0};
  }
  for (int j0 = 0; j0 < n; j0 += 4 * kEbcBatch) {
    EbcBatch<TIn> nxt;
    const bool more = j0 + 4 * kEbcBatch < n;
    ebc_load<TIn, kUnit>(nxt, more ? t : next, L, more ? j0 + 4 * kEbcBatch : 0);
    if (kUnit && j0 + 4 * kEbcBatch > n) {  // the last elements of a unit line: j = j0 + g and every fourth
#pragma unroll
      for (int m = 0; m < M; ++m) {
        idx[m] = (int)((uint32_t)(step[m] * (j0 + g)) % (uint32_t)n);
        step[m] = ebc_wrap(4 * step[m], n);
      }
    }
#pragma unroll
    for (int u = 0; u < kEbcBatch; ++u) {
      if (j0 + 4 * u >= n) break;  // uniform
      double b[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        b[c] = (double)cur.v[u][c];
        if constexpr (kSumIn) e_in = fma(b[c], b[c], e_in);
      }
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const double a = tab[part[m] + idx[m]];
        idx[m] += step[m];
        if (idx[m] >= n) idx[m] -= n;
#pragma unroll
        for (int c = 0; c < 2; ++c) acc[m][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[c], acc[m][c], 0, 0, 0);
      }
    }
    if constexpr (kUnit) {
#pragma unroll
      for (int m = 0; m < M; ++m) idx[m] = ebc_wrap(ebc_wrap(ebc_wrap(idx[m] + 12 * step[m], n), n), n);  // (12 f <= 3 n)
    }
    cur = nxt;
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const long long col = t.col0 + 16 * c + l16;
    double w = 1.0;  // weight of the line
    if (L.wdiv) {
      const long long c1 = ebc_div(col, L.wdiv), ky = ebc_div(c1, L.wmod);
      w = (ky > 0 ? 2.0 : 1.0) * (c1 - ky * L.wmod > 0 ? 2.0 : 1.0);
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int k = (kt + m) * 16 + g + 4 * r;
        if (k < K && t.ok[c]) {
          const double v = acc[m][c][r];
          e_out = fma((k > 0 ? 2.0 : 1.0) * w * v, v, e_out);
          if constexpr (kStore) out[(long long)k * L.lines + col] = v;
        }
      }
  }
}

// All coefficients of the lines workgroup `blk` of `n_blk` owns; e_out += weighted sum of their
// squares, e_in += sum of the squares of the elements (kSumIn).  The loads of the next 16 elements,
// or of the next tile, are always in flight, those of the first while the table is made: a line is
// short, and a wavefront that waited for every load would do nothing else.
// A unit of work is a tile of lines, or (kShared) every share-th pair of its coefficient tiles.
template <bool kShared, typename TIn, bool kUnit, bool kStore, bool kSumIn>
__device__ __forceinline__ void ebc_contract(const TIn *__restrict__ in, double *__restrict__ out,
                                             const EbcLines &L, int blk, int n_blk, double *tab,
                                             double &e_out, double &e_in) {
  const int wave = threadIdx.x >> 6;
  const int K = ebc_coefs(L.n), KT = (K + 15) / 16, share = kShared ? L.share : 1;
  const long long units = (L.lines + kEbcTileCols - 1) / kEbcTileCols * share;
  const long long first = (long long)blk * kEbcWaves + wave, stride = (long long)n_blk * kEbcWaves;
  auto tile_of = [&](long long u) -> long long { return kShared ? ebc_div(u, share) : u; };
  EbcTile<TIn> t = ebc_tile_at<TIn, kUnit>(in, L, tile_of(first));
  EbcBatch<TIn> cur;
  ebc_load<TIn, kUnit>(cur, t, L, 0);
  ebc_table(L.n, tab);
  for (long long u = first; u < units; u += stride) {
    const EbcTile<TIn> next = ebc_tile_at<TIn, kUnit>(in, L, tile_of(u + stride));  // (past the end: no line exists)
    int kt = kShared ? 2 * (int)(u - tile_of(u) * share) : 0;
    auto after = [&](int k) -> const EbcTile<TIn> & { return k < KT ? t : next; };
    if (KT == 1) {
      ebc_tile<1, TIn, kUnit, kStore, kSumIn>(cur, t, next, out, L, tab, 0, K, e_out, e_in);
    } else {
      if (kt == 0) {
        ebc_tile<2, TIn, kUnit, kStore, kSumIn>(cur, t, after(2 * share), out, L, tab, 0, K, e_out, e_in);
        kt = 2 * share;
      }
      for (; kt < KT; kt += 2 * share) {
        if (kt + 1 < KT)
          ebc_tile<2, TIn, kUnit, kStore, false>(cur, t, after(kt + 2 * share), out, L, tab, kt, K, e_out, e_in);
        else
          ebc_tile<1, TIn, kUnit, kStore, false>(cur, t, after(kt + 2 * share), out, L, tab, kt, K, e_out, e_in);
      }
    }
    t = next;
  }
}

// Tickets: atomics on one address are served one after another, some 35 ns each, which is 14 us with 400 workgroups and 30
// with 864.  So a workgroup draws from one of 32 leaves (cache lines of their own), and the last of each leaf from the
// root.  They lie in the halves of the partial sums that the first launch leaves unused, which zeroes them.
constexpr int kEbcLeaves = 32, kEbcTicketLine = 16;  // (doubles)
__host__ __device__ __forceinline__ unsigned *ebc_leaf(double *partials, int i) {
  return reinterpret_cast<unsigned *>(partials + kEbcPartials / 2 + i * kEbcTicketLine);
}
__host__ __device__ __forceinline__ unsigned *ebc_root(double *partials) {
  return reinterpret_cast<unsigned *>(partials + kEbcPartials + kEbcPartials / 2);
}
static_assert(kEbcLeaves * kEbcTicketLine <= kEbcPartials / 2, "room of the tickets");

// Workgroups [0, gx): x coefficients of err -> cx, |err|^2.  [gx, gx + gt): S_T of err.  The rest:
// |dense|^2.  The tickets of the last launch are zeroed.
template <bool kShared>
__global__ __launch_bounds__(kEbcThreads, 4) void ebc_first_kernel(
    const float *__restrict__ err, const float *__restrict__ dense, long long total, EbcLines lx, EbcLines lt,
    int gx, int gt, double *__restrict__ cx, double *__restrict__ partials) {
  __shared__ double tab[2 * kEbcMaxAxis];
  __shared__ double red[kEbcWaves];
  int blk = blockIdx.x;
  double e_out = 0.0, e_in = 0.0;
  if (blk < gx) {
    ebc_contract<kShared, float, true, true, true>(err, cx, lx, blk, gx, tab, e_out, e_in);
    // (e_in of a line is spread over the four lane groups, each element once)
    const double s = ebc_block_sum(e_in, red);
    if (threadIdx.x == 0) {
      partials[0 * kEbcPartials + blk] = s;
      if (blk == 0) *ebc_root(partials) = 0u;
    }
    if (blk == 0 && threadIdx.x < kEbcLeaves) *ebc_leaf(partials, (int)threadIdx.x) = 0u;
  } else if (blk < gx + gt) {
    blk -= gx;
    ebc_contract<kShared, float, false, false, false>(err, nullptr, lt, blk, gt, tab, e_out, e_in);
    const double s = ebc_block_sum(e_out, red);
    if (threadIdx.x == 0) partials[1 * kEbcPartials + blk] = s;
  } else {
    blk -= gx + gt;
    const long long stride = (long long)(gridDim.x - gx - gt) * kEbcThreads, t0 = (long long)blk * kEbcThreads + threadIdx.x;
    constexpr int U = 8;  // loads in flight
    const bool wide = (reinterpret_cast<uintptr_t>(dense) & 15u) == 0;
    const long long quads = wide ? total / 4 : 0;
    const float4 *dense4 = reinterpret_cast<const float4 *>(dense);
    for (long long e = t0; e < quads; e += U * stride) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = e + u * stride < quads ? dense4[e + u * stride] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < U; ++u)
        e_in = fma((double)v[u].w, (double)v[u].w,
                   fma((double)v[u].z, (double)v[u].z, fma((double)v[u].y, (double)v[u].y, fma((double)v[u].x, (double)v[u].x, e_in))));
    }
    for (long long e = 4 * quads + t0; e < total; e += stride) e_in = fma((double)dense[e], (double)dense[e], e_in);
    const double s = ebc_block_sum(e_in, red);
    if (threadIdx.x == 0) partials[4 * kEbcPartials + blk] = s;
  }
}

// y coefficients of the x coefficients -> cyx, S_XY
template <bool kShared>
__global__ __launch_bounds__(kEbcThreads, 3) void ebc_second_kernel(const double *__restrict__ cx, EbcLines ly,
                                                                 double *__restrict__ cyx,
                                                                 double *__restrict__ partials) {
  __shared__ double tab[2 * kEbcMaxAxis];
  __shared__ double red[kEbcWaves];
  double e_out = 0.0, e_in = 0.0;
  ebc_contract<kShared, double, true, true, false>(cx, cyx, ly, blockIdx.x, gridDim.x, tab, e_out, e_in);
  const double s = ebc_block_sum(e_out, red);
  if (threadIdx.x == 0) partials[2 * kEbcPartials + blockIdx.x] = s;
}

struct EbcFinish {
  int count[kEbcSums];  // partial sums of each reduction
  double n_t, n_yx, w[4], epsilon;
};

// Ends a launch: this workgroup's sum of reduction 3 is `s` (and of reduction 2 `s_xy`, if kBoth); the workgroup that
// draws the last ticket adds up all partial sums and writes the result.  The partial sums of this launch cross
// workgroups of different XCDs and therefore move with device-scope stores and loads; a workgroup takes its
// ticket after its stores are acknowledged.
template <bool kBoth>
__device__ __forceinline__ void ebc_finish(double s_xy, double s, double *__restrict__ partials, const EbcFinish &f,
                                           double *__restrict__ out) {
  __shared__ int s_last;
  if (threadIdx.x == 0) {
    if constexpr (kBoth)
      __hip_atomic_store(&partials[2 * kEbcPartials + blockIdx.x], s_xy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&partials[3 * kEbcPartials + blockIdx.x], s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    const int leaf = (int)(blockIdx.x % kEbcLeaves), n_leaves = min((int)gridDim.x, kEbcLeaves);
    const unsigned members = (gridDim.x - (unsigned)leaf + kEbcLeaves - 1) / kEbcLeaves;
    bool last = atomicAdd(ebc_leaf(partials, leaf), 1u) == members - 1;
    if (last) last = atomicAdd(ebc_root(partials), 1u) == (unsigned)n_leaves - 1;
    s_last = last;
  }
  __syncthreads();
  if (!s_last) return;
  double v[kEbcSums][kEbcPartials / kEbcThreads];
#pragma unroll
  for (int k = 0; k < kEbcSums; ++k)
#pragma unroll
    for (int u = 0; u < kEbcPartials / kEbcThreads; ++u) {
      const int i = threadIdx.x + u * kEbcThreads;
      v[k][u] = i < f.count[k] ? __hip_atomic_load(&partials[k * kEbcPartials + i], __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT)
                               : 0.0;
    }
  __shared__ double fin[kEbcSums][kEbcWaves];
#pragma unroll
  for (int k = 0; k < kEbcSums; ++k) {
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < kEbcPartials / kEbcThreads; ++u) a += v[k][u];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) a += __shfl_xor(a, d, 64);
    if ((threadIdx.x & 63) == 0) fin[k][threadIdx.x >> 6] = a;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double sums[kEbcSums];
#pragma unroll
    for (int k = 0; k < kEbcSums; ++k) sums[k] = (fin[k][0] + fin[k][1]) + (fin[k][2] + fin[k][3]);
    const double n_tot = f.n_t * f.n_yx;
    const double a = f.n_yx * sums[1], b = f.n_t * sums[2], ll = sums[3];
    const double lh = a - ll, hl = b - ll, hh = n_tot * sums[0] - a - b + ll;
    out[0] = (f.w[0] * ll + f.w[1] * lh + f.w[2] * hl + f.w[3] * hh) / (n_tot * sums[4] + f.epsilon);
    out[1] = ll;
    out[2] = lh;
    out[3] = hl;
    out[4] = hh;
    out[5] = n_tot * sums[4];
  }
}

// S_XYT
template <bool kShared>
__global__ __launch_bounds__(kEbcThreads, 3) void ebc_third_kernel(const double *__restrict__ cyx, EbcLines lt,
                                                                double *__restrict__ partials, EbcFinish f,
                                                                double *__restrict__ out) {
  __shared__ double tab[2 * kEbcMaxAxis];
  __shared__ double red[kEbcWaves];
  double e_out = 0.0, e_in = 0.0;
  ebc_contract<kShared, double, true, false, false>(cyx, nullptr, lt, blockIdx.x, gridDim.x, tab, e_out, e_in);
  ebc_finish<false>(0.0, ebc_block_sum(e_out, red), partials, f, out);
}

// The second and third step in one launch, for short t and y axes (latents have 21 to 33 and 30 to 45): a wavefront
// takes a (t, y) plane of one x coefficient of one channel, contracts y and then t, and keeps
// nothing but the two sums of squares.  With the plane's rows as the first operand and the table as the second the y
// coefficients come out as (t = lane / 16 + 4 r, k = lane % 16) in register r, which is, unchanged, the second operand
// of the t contraction's step r.  The table's operands over y stay in registers.  Bound by latency as the others: one
// plane a wavefront at 128 x 21 x 30 x 52, 13 us (14.7 under the profiler) in the place of two launches of 10 and 13 us and
// of 10 MB written and read again (21 us with one ticket for its 864 workgroups and operands from LDS in every step).
// Longest axes: two tiles of 16 coefficients over t; over y what the registers of a wavefront hold (16 steps took 35 of them to
// scratch).  Whole call, three launches -> two, T = 3 to 63, X = 52: Y = 8 to 45 4 to 30 % faster at 16 and at 128 channels (16 x
// 63 x 45 33.0 -> 30.8 us, 128 x 34 x 45 81.6 -> 78.7), Y = 49 to 63 up to 17 % slower (16 x 63 x 49 34.0 -> 40.0, 128 x 33 x 56
// 85 -> 98).
constexpr int kEbcPlaneT = 63, kEbcPlaneY = 48;
template <int M, int SY>  // tiles of y coefficients, contraction steps (of 4 elements) over y
__global__ __launch_bounds__(kEbcThreads, SY > 8 ? 3 : 4) void ebc_plane_kernel(const double *__restrict__ cx, int C, int T, int Y,
                                                                                int KX, double *__restrict__ partials,
                                                                                EbcFinish f, double *__restrict__ out) {
  __shared__ double tab_t[2 * kEbcPlaneT], tab_y[2 * kEbcPlaneY];
  __shared__ double red[kEbcWaves];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, g = lane >> 4;
  const int KY = ebc_coefs(Y), KT = ebc_coefs(T), PT = (KT + 15) / 16, TT = (T + 15) / 16, TY = T * Y;
  const long long planes = (long long)KX * C, stride = (long long)gridDim.x * kEbcWaves;
  long long p = (long long)blockIdx.x * kEbcWaves + wave;
  // row l16 of t tile tt of plane pl, this lane's element of each step
  auto load = [&](double (&v)[SY], long long pl, int tt) __attribute__((always_inline)) {
    const int t = 16 * tt + l16;
    const double *src = cx + pl * TY + t * Y + g;
    const int last = pl < planes && t < T ? Y - g : 0;
#pragma unroll
    for (int u = 0; u < SY; ++u) v[u] = 4 * u < last ? src[4 * u] : 0.0;
  };
  double cur[SY];
  load(cur, p, 0);
  for (int m = threadIdx.x; m < T + Y; m += kEbcThreads) {  // (tables as ebc_table's)
    const int n = m < T ? T : Y, i = m < T ? m : m - T;
    double *tab = m < T ? tab_t : tab_y;
    double c, sn;
    sincospi(2.0 * (double)i / (double)n, &sn, &c);
    tab[i] = c;
    tab[n + i] = sn;
  }
  __syncthreads();
  // this lane's coefficient of each tile: (f j) mod n at its first j, the step for j + 4, the half of the table
  struct Walk { int at, step, half; };
  auto walk = [&](int k, int K, int n) -> Walk {
    const int fr = k < K ? (k + 1) >> 1 : 0;  // (coefficients past K are computed and dropped)
    return Walk{(int)((uint32_t)(fr * g) % (uint32_t)n), (int)((uint32_t)(4 * fr) % (uint32_t)n), (k & 1) == 0 && k > 0 && k < K ? n : 0};
  };
  double by[M][SY];  // the table's operands of all steps over y
#pragma unroll
  for (int m = 0; m < M; ++m) {
    Walk w = walk(16 * m + l16, KY, Y);
#pragma unroll
    for (int u = 0; u < SY; ++u) {
      by[m][u] = tab_y[w.half + w.at];
      w.at += w.step;
      w.at -= w.at >= Y ? Y : 0;
    }
  }
  Walk wt[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) wt[q] = walk(16 * q + l16, KT, T);
  double s_xy = 0.0, s_xyt = 0.0;
  for (; p < planes; p += stride) {
    const double wx = p >= C ? 2.0 : 1.0;  // (plane = kx * C + channel)
    ebc_f64x4 acc2[M][2];
    int at_t[2] = {wt[0].at, wt[1].at};
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int q = 0; q < 2; ++q) acc2[m][q] = ebc_f64x4{0.0, 0.0, 0.0, 0.0};
    for (int tt = 0; tt < TT; ++tt) {
      double nxt[SY];
      const bool same = tt + 1 < TT;
      load(nxt, same ? p : p + stride, same ? tt + 1 : 0);
      ebc_f64x4 acc[M];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        acc[m] = ebc_f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < SY; ++u) acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(cur[u], by[m][u], acc[m], 0, 0, 0);
      }
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int ky = 16 * m + l16;
        const double w = ky > 0 ? 2.0 * wx : wx;
        // (coefficients past KY are left out, not weighted with 0: they are infinite with an infinite element; rows past T are zero)
        if (ky < KY)
#pragma unroll
          for (int r = 0; r < 4; ++r) s_xy = fma(w * acc[m][r], acc[m][r], s_xy);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (q >= PT) break;  // uniform
        double a[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          a[r] = tab_t[wt[q].half + at_t[q]];
          at_t[q] += wt[q].step;
          at_t[q] -= at_t[q] >= T ? T : 0;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int m = 0; m < M; ++m) acc2[m][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[r], acc[m][r], acc2[m][q], 0, 0, 0);
      }
#pragma unroll
      for (int u = 0; u < SY; ++u) cur[u] = nxt[u];
    }
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int ky = 16 * m + l16;
      const double w = ky > 0 ? 2.0 * wx : wx;
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int kt = 16 * q + g + 4 * r;
          const double v = acc2[m][q][r];
          if (ky < KY && kt < KT) s_xyt = fma((kt > 0 ? 2.0 : 1.0) * w * v, v, s_xyt);
        }
    }
  }
  const double sum_xy = ebc_block_sum(s_xy, red);
  const double sum = ebc_block_sum(s_xyt, red);
  ebc_finish<true>(sum_xy, sum, partials, f, out);
}

// the two coefficient arrays (neither larger than the tensor), the partial sums with the tickets
static size_t ebc_workspace_doubles(long long total, int T, int Y, int X) {
  return 2 * (size_t)total + (size_t)(T + Y + X) + kEbcSums * (size_t)kEbcPartials;
}

int launch_ebc_band_error(long long C, int T, int Y, int X, const float *err, const float *dense,
                          const double *w, double epsilon, double *ws, double *out,
                          hipStream_t st) {
  const long long total = C * T * Y * X;
  const int KX = ebc_coefs(X), KY = ebc_coefs(Y);
  double *cx = ws, *cyx = cx + total, *partials = cyx + total;
  EbcLines lx{X, 1, C * T * Y, 0, 1, 1};
  EbcLines lt{T, (long long)Y * X, C * Y * X, 0, 1, 1};
  EbcLines ly{Y, 1, (long long)KX * C * T, C * T, KX, 1};
  EbcLines lyx{T, 1, (long long)KY * KX * C, C, KX, 1};
  // workgroups of a contraction: one tile per wavefront, or the fewest equal rounds that leave no
  // more than `most`: the workgroups of a launch are resident at once (four wavefronts per SIMD in
  // the first, where the three parts share them by their matrix work and bytes at 21 x 30 x 52; three
  // in the others).  With at most a quarter as many tiles as wavefronts the coefficients of a tile are dealt over
  // as many as there are for it: a long axis and few lines would else leave one wavefront hundreds of
  // coefficients of hundreds of elements (1 x 5 x 9 x 1000: 912 -> 83 us, 16 x 1024 x 8 x 8: 2003 -> 169 us;
  // with half as many tiles, 16 x 33 x 45 x 80: 37.5 -> 38.7 us).
  auto groups = [](EbcLines &l, long long most) -> int {
    const long long tiles = (l.lines + kEbcTileCols - 1) / kEbcTileCols, places = most * kEbcWaves / tiles;
    const int pairs = ((ebc_coefs(l.n) + 15) / 16 + 1) / 2;
    if (places >= 4) l.share = places < pairs ? (int)places : pairs;
    const long long g = (tiles * l.share + kEbcWaves - 1) / kEbcWaves;
    const long long rounds = (g + most - 1) / most;
    return (int)((g + rounds - 1) / rounds);
  };
  const int gx = groups(lx, 384), gt = groups(lt, 400);
  const int gd = (int)std::min<long long>((total + 8 * kEbcThreads - 1) / (8 * kEbcThreads), 240);
  EbcFinish f{{gx, gt, 0, 0, gd}, (double)T, (double)Y * X, {w[0], w[1], w[2], w[3]}, epsilon};
  auto first = lx.share > 1 || lt.share > 1 ? ebc_first_kernel<true> : ebc_first_kernel<false>;
  hipLaunchKernelGGL(first, dim3((unsigned)(gx + gt + gd)), dim3(kEbcThreads), 0, st, err, dense, total, lx, lt, gx, gt, cx,
                     partials);
  if (T <= kEbcPlaneT && Y <= kEbcPlaneY && C <= 0x7fffffff / KX) {
    const long long want = ((long long)KX * C + kEbcWaves - 1) / kEbcWaves;
    const int gp = (int)std::min<long long>(want, kEbcPartials);
    f.count[2] = f.count[3] = gp;
    auto plane = Y < 32 ? ebc_plane_kernel<1, 8> : ebc_plane_kernel<2, 12>;
    hipLaunchKernelGGL(plane, dim3((unsigned)gp), dim3(kEbcThreads), 0, st, cx, (int)C, T, Y, KX, partials, f, out);
    return check_launch("ebc kernels");
  }
  const int gy = groups(ly, 768), gyx = groups(lyx, 768);
  f.count[2] = gy;
  f.count[3] = gyx;
  auto second = ly.share > 1 ? ebc_second_kernel<true> : ebc_second_kernel<false>;
  auto third = lyx.share > 1 ? ebc_third_kernel<true> : ebc_third_kernel<false>;
  hipLaunchKernelGGL(second, dim3((unsigned)gy), dim3(kEbcThreads), 0, st, cx, ly, cyx, partials);
  hipLaunchKernelGGL(third, dim3((unsigned)gyx), dim3(kEbcThreads), 0, st, cyx, lyx, partials, f, out);
  return check_launch("ebc kernels");
}

// ---------------------------------------------------------------------------------------
// Selection (host).  Heads i = 0..n-1, candidates c = 0..k-1 with error E[i*k+c] and
// sparsity S[i*k+c]; minimise sum E subject to sum S >= need.
namespace {

struct Inc {       // one step along a head's lower convex hull
  int head, to;    // candidate reached by taking this step (and all earlier ones of the head)
  double ds, de;   // gain in sparsity (> 0) and cost in error (>= 0 after dominance pruning)
};

struct Solver {
  int n, k;
  const double *E, *S;
  double need;
  std::vector<int> base;               // per head: candidate of least error (ties: most sparse)
  std::vector<std::vector<int>> hull;  // per head: hull candidates after base, sparsity ascending
  std::vector<Inc> incs;               // all hull steps, cheapest error per sparsity first
  std::vector<int> fixed, best;
  std::vector<char> removed;           // [n*k] candidates proved useless by their reduced cost
  double best_e;
  long long nodes;

  double e(int i, int c) const { return E[(size_t)i * k + c]; }
  double s(int i, int c) const { return S[(size_t)i * k + c]; }

  bool ok(int i, int c) const { return !removed[(size_t)i * k + c]; }

  void build() {
    base.assign(n, 0);
    hull.assign(n, {});
    incs.clear();
    for (int i = 0; i < n; ++i) {
      int b = -1;
      for (int c = 0; c < k; ++c)
        if (ok(i, c) && (b < 0 || e(i, c) < e(i, b) || (e(i, c) == e(i, b) && s(i, c) > s(i, b)))) b = c;
      base[i] = b;  // (at least one candidate of every head survives the reduction)
      // candidates that add sparsity over the base, by sparsity; keep the lower convex hull
      std::vector<int> cand;
      for (int c = 0; c < k; ++c)
        if (ok(i, c) && s(i, c) > s(i, b)) cand.push_back(c);
      std::sort(cand.begin(), cand.end(), [&](int a, int c2) {
        return s(i, a) < s(i, c2) || (s(i, a) == s(i, c2) && e(i, a) < e(i, c2));
      });
      std::vector<int> h = {b};
      for (int c : cand) {
        if (s(i, c) == s(i, h.back())) continue;  // same sparsity, more error
        while (h.size() >= 2) {
          const int p1 = h[h.size() - 2], p2 = h.back();
          // drop p2 if it lies on or above the segment p1 -> c
          const double cross = (s(i, p2) - s(i, p1)) * (e(i, c) - e(i, p1)) -
                               (e(i, p2) - e(i, p1)) * (s(i, c) - s(i, p1));
          if (cross <= 0.0) h.pop_back(); else break;
        }
        h.push_back(c);
      }
      for (size_t j = 1; j < h.size(); ++j) {
        hull[i].push_back(h[j]);
        incs.push_back({i, h[j], s(i, h[j]) - s(i, h[j - 1]), e(i, h[j]) - e(i, h[j - 1])});
      }
    }
    std::stable_sort(incs.begin(), incs.end(),
                     [](const Inc &a, const Inc &b) { return a.de * b.ds < b.de * a.ds; });
  }

  // Relaxation with some heads fixed.  Returns the bound; `frac_head` is the head whose step
  // was taken partially (-1 if the relaxed solution is integral), `sol` the integral part.
  bool relax(double &bound, int &frac_head, std::vector<int> &sol, double &sol_e, double &sol_s,
             double *lambda = nullptr) {
    double se = 0.0, ss = 0.0;
    sol.assign(n, 0);
    for (int i = 0; i < n; ++i) {
      sol[i] = fixed[i] >= 0 ? fixed[i] : base[i];
      se += e(i, sol[i]);
      ss += s(i, sol[i]);
    }
    frac_head = -1;
    if (lambda) *lambda = 0.0;
    if (ss >= need) { bound = se; sol_e = se; sol_s = ss; return true; }
    for (const Inc &in : incs) {
      if (fixed[in.head] >= 0) continue;
      if (ss + in.ds >= need) {
        // this step reaches the budget: fractional unless it lands exactly on it
        const double f = (need - ss) / in.ds;
        bound = se + f * in.de;
        frac_head = in.head;
        if (lambda) *lambda = in.de / in.ds;
        // integral completion: take the whole step (feasible)
        sol[in.head] = in.to;
        sol_e = se + in.de;
        sol_s = ss + in.ds;
        return true;
      }
      sol[in.head] = in.to;
      se += in.de;
      ss += in.ds;
    }
    return false;  // budget out of reach
  }

  // Single-head moves that lower the error and keep the budget, best first, until none is left.
  void improve(std::vector<int> &sol, double &sol_e, double &sol_s) const {
    for (;;) {
      int bi = -1, bc = -1;
      double gain = 0.0;
      for (int i = 0; i < n; ++i) {
        if (fixed[i] >= 0) continue;
        const double e0 = e(i, sol[i]), s0 = s(i, sol[i]);
        for (int c = 0; c < k; ++c) {
          if (!ok(i, c)) continue;
          const double de = e0 - e(i, c);
          if (de > gain && sol_s - s0 + s(i, c) >= need) gain = de, bi = i, bc = c;
        }
      }
      if (bi < 0) return;
      sol_e -= gain;
      sol_s += s(bi, bc) - s(bi, sol[bi]);
      sol[bi] = bc;
    }
  }

  static constexpr long long kNodeLimit = 2000000;
  void search() {
    if (++nodes > kNodeLimit) return;
    double bound, se, ss;
    int fh;
    std::vector<int> sol;
    if (!relax(bound, fh, sol, se, ss)) return;
    if (bound >= best_e) return;
    if (se < best_e + (best_e - bound)) improve(sol, se, ss);  // worth polishing
    if (se < best_e) { best_e = se; best = sol; }  // the integral completion is feasible
    if (fh < 0 || bound >= best_e) return;          // relaxed solution was integral
    // branch on the fractional head: each of its candidates in turn, most promising first
    std::vector<int> order(k);
    for (int c = 0; c < k; ++c) order[c] = c;
    std::sort(order.begin(), order.end(), [&](int a, int b) { return e(fh, a) < e(fh, b); });
    for (int c : order) {
      if (!ok(fh, c)) continue;
      fixed[fh] = c;
      search();
    }
    fixed[fh] = -1;
  }
};

}  // namespace

int ebc_select_host(int n, int k, const double *E, const double *S, double s_min, int *choice,
                    double *total_error, long long *nodes) {
  Solver sv;
  sv.n = n; sv.k = k; sv.E = E; sv.S = S;
  sv.need = s_min * (double)n - 1e-12 * (double)n;
  sv.removed.assign((size_t)n * k, 0);
  sv.build();
  sv.fixed.assign(n, -1);
  sv.best_e = INFINITY;
  sv.nodes = 0;
  {
    // Root: relaxation, incumbent, and reduced-cost fixing.  With the multiplier lambda of
    // the relaxation, any selection that uses candidate (i, c) costs at least
    //   bound + (E_ic - lambda S_ic) - min_c' (E_ic' - lambda S_ic'),
    // so candidates for which that is not below the incumbent can be discarded.  The gap of
    // this problem is at most one hull step, so almost every head is left with one candidate.
    double bound, se, ss, lambda;
    int fh;
    std::vector<int> sol;
    if (sv.relax(bound, fh, sol, se, ss, &lambda)) {
      sv.improve(sol, se, ss);
      sv.best_e = se;
      sv.best = sol;
      if (fh >= 0) {
        const double gap = se - bound;
        for (int i = 0; i < n; ++i) {
          double lo = INFINITY;
          for (int c = 0; c < k; ++c) lo = std::min(lo, sv.e(i, c) - lambda * sv.s(i, c));
          for (int c = 0; c < k; ++c)
            if (sv.e(i, c) - lambda * sv.s(i, c) - lo >= gap + 1e-15 * std::fabs(se) && c != sol[i])
              sv.removed[(size_t)i * k + c] = 1;
        }
        sv.build();
        sv.search();
      }
    }
  }
  if (nodes) *nodes = sv.nodes;
  if (sv.best.empty()) return 1;  // infeasible
  if (sv.nodes > Solver::kNodeLimit) return 2;  // optimality not proved within the node limit
  for (int i = 0; i < n; ++i) choice[i] = sv.best[i];
  double tot = 0.0;
  for (int i = 0; i < n; ++i) tot += sv.e(i, sv.best[i]);
  *total_error = tot;
  return 0;
}

size_t ebc_workspace_bytes(long long C, int T, int Y, int X) {
  return ebc_workspace_doubles(C * T * Y * X, T, Y, X) * sizeof(double);
}

}  // namespace heart
