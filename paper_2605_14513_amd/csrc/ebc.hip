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
//    accumulators and reduced in a fixed order.  One launch and the total where its workgroups fill the chip once (ebc_one_launch):
//      ebc_channel everything: a channel's planes from the tensor to S_XY and S_XYT, |err|^2 and S_T, |dense|^2 in its workgroups
//      ebc_total  one workgroup adds up
//    or two launches with the x coefficients between them:
//      ebc_first  x coefficients of err with |err|^2, S_T of err, |dense|^2
//      ebc_plane  y and t coefficients of the x coefficients with S_XY and S_XYT; its last workgroup adds everything up
//    or, where t is longer than 63 or y than 48, in the place of the second
//      ebc_second y coefficients of the x coefficients with S_XY
//      ebc_third  S_XYT; its last workgroup adds everything up
//    Bound by latency and, with many channels, the bytes of err and dense: 128 x 21 x 30 x 52 33.1 -> 21.4 us with one launch (15 us
//    of it the planes: 3 until the operands are there, 2.5 a plane, 1.3 over t; 18 the lines of S_T beside them and |dense|^2), of
//    which the matrix instructions are 3 and the bytes 6 to 8.  Before: 41.6 us with three launches that counted
//    400 workgroups on one ticket, 257 with twelve that convolved in fp64 on the vector units (results equal to 1e-15).
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
template <int kThreads = kEbcThreads>
__device__ __forceinline__ void ebc_table(int n, double *tab) {
  for (int m = threadIdx.x; m < n; m += kThreads) {
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

// this thread's sum of squares of a tensor, workgroup `blk` of `n_blk`
template <int kThreads>
__device__ __forceinline__ double ebc_squares(const float *__restrict__ dense, long long total, int blk, int n_blk) {
  double e_in = 0.0;
  const long long stride = (long long)n_blk * kThreads, t0 = (long long)blk * kThreads + threadIdx.x;
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
  return e_in;
}

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
    e_in = ebc_squares<kEbcThreads>(dense, total, blk, (int)gridDim.x - gx - gt);
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

// The result from all partial sums, by one workgroup.  (Device-scope loads: see ebc_finish.)
__device__ __forceinline__ void ebc_total(double *__restrict__ partials, const EbcFinish &f, double *__restrict__ out) {
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
  ebc_total(partials, f, out);
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

// All contractions of short axes in one launch (a second, of one workgroup, adds up).
// S_XY, S_XYT: a workgroup takes the planes (t) of one channel and 16 of the x coefficients, a wavefront a plane at a
// time.  Cosines are even and sines are odd about the middle of the axis, so the coefficients of a row are those of the sums e_j +
// e_(X-j), j <= X / 2, against cosines and of the differences against sines: half the elements, and a group of 16 coefficients is
// of one kind.  With the plane's rows as the first operand and the table as the second, the x coefficients come out
// as (y = lane / 16 + 4 r, k = lane % 16) in register r, which is, unchanged, the second operand of the y contraction's step r: a
// plane goes from the tensor to its y-x coefficients in registers.  The coefficients of all planes meet in LDS, 16 *
// (2 (Y / 4) + 1) doubles a plane, where the wavefronts contract over t.  No coefficient goes through memory; err is read once for
// each group of 16, from the L2 of the channel's XCD, and once for S_T.  Sums and differences of two floats are as good as exact in
// fp64 (error of the energies against a transform in 64 bits 1e-16 of their sum, as before).
// S_T, |err|^2: a thread takes lines, sums and differences as above, on the vector units (a line has few coefficients: tiles of 16 would be
// half empty, and the matrix units are what the planes wait for).
// Workgroups [0, n_ch): the planes.  [n_ch, n_ch + gt): S_T and |err|^2.  The rest: |dense|^2.
constexpr int kEbcChThreads = 512, kEbcChWaves = kEbcChThreads / 64;
constexpr int kEbcChLds = 144 * 1024;  // room for the largest sizes that it holds (T = 35, Y = 48, X = 95)

// a mod n for 0 <= a < 2^16, rn = 1 / n
__device__ __forceinline__ int ebc_mod(int a, int n, float rn) {
  const int r = a - (int)((float)a * rn) * n;  // (the quotient may be one off)
  return r < 0 ? r + n : r >= n ? r - n : r;
}

// sum over the wavefront in every lane, on the vector units (through LDS, as __shfl does it, three sums took 0.8 us)
__device__ __forceinline__ double ebc_wave_sum(double v) {
  auto halves = [](double x, uint32_t &lo, uint32_t &hi) {
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    lo = (uint32_t)u;
    hi = (uint32_t)(u >> 32);
  };
  auto whole = [](uint32_t lo, uint32_t hi) -> double { return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo); };
  uint32_t lo, hi;
#define HEART_EBC_DPP(ctrl)                                                     \
  halves(v, lo, hi);                                                            \
  v += whole(__builtin_amdgcn_update_dpp(0u, lo, ctrl, 0xf, 0xf, false),        \
             __builtin_amdgcn_update_dpp(0u, hi, ctrl, 0xf, 0xf, false))
  HEART_EBC_DPP(0xB1);   // quad_perm, lane ^ 1
  HEART_EBC_DPP(0x4E);   // quad_perm, lane ^ 2
  HEART_EBC_DPP(0x124);  // row_ror:4
  HEART_EBC_DPP(0x128);  // row_ror:8
#undef HEART_EBC_DPP
  uint32_t l0, l1, h0, h1;
  halves(v, lo, hi);
  swap_rows16(lo, l0, l1);
  swap_rows16(hi, h0, h1);
  v = whole(l0, h0) + whole(l1, h1);
  halves(v, lo, hi);
  swap_halves32(lo, l0, l1);
  swap_halves32(hi, h0, h1);
  return whole(l0, h0) + whole(l1, h1);
}

// S_T and the sum of squares of the lines of this thread; coefficients up to frequency R >= T / 4, P >= T / 2 pairs.  Behind the table
// of T in LDS the factors of the pairs, [P][2 R + 2].  All elements of a line are asked for at once, those of the next
// line as soon as a register is free.  (No branches: loads that may not be there are all waited for.)
template <int R, int P>
__device__ __forceinline__ void ebc_lines_t(const float *__restrict__ err, long long lines, int T, int inner, int blk, int n_blk,
                                            double *tab, double &s_t, double &s_in) {
  constexpr int K = 2 * R + 2;
  const int r = T / 4, pairs = T / 2;  // (the middle of an even T is a pair without a second element)
  const uint32_t bytes = (uint32_t)(4 * lines * T);
  float e0, a[P], b[P];
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(err), 0, (int)bytes, 0x00020000);
  uint32_t at;  // byte offset of the line
  auto seek = [&](long long l) __attribute__((always_inline)) {
    const uint32_t l32 = (uint32_t)min(l, lines - 1), o = l32 / (uint32_t)inner;  // (a line past the end is not counted)
    at = 4u * (o * (uint32_t)(T * inner) + (l32 - o * (uint32_t)inner));
  };
  // (an element that does not exist is out of range for the descriptor and arrives as zero)
  auto element = [&](int t, bool there) __attribute__((always_inline)) -> float {
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, there ? at + (uint32_t)(4 * t * inner) : 0xffffffffu, 0, 0));
  };
  auto ask = [&](int u) __attribute__((always_inline)) {  // pair u: elements u + 1 and T - 1 - u
    a[u] = element(u + 1, u < pairs);
    b[u] = element(T - 1 - u, u < pairs && 2 * (u + 1) != T);
  };
  const long long stride = (long long)n_blk * kEbcChThreads;
  long long l0 = (long long)blk * kEbcChThreads + threadIdx.x;
  seek(l0);
  e0 = element(0, true);
#pragma unroll
  for (int u = 0; u < P; ++u) ask(u);
  ebc_table<kEbcChThreads>(T, tab);
  // row t - 1: cosines of f = 0 .. R at t, sines of f = 1 .. R
  double *op = tab + 2 * T;
  for (int i = threadIdx.x; i < P * K; i += kEbcChThreads) {
    const int t = i / K + 1, k = i % K, f = k <= R ? k : k - R;
    op[i] = k < K - 1 && f <= r ? tab[(k <= R ? 0 : T) + ebc_mod(f * t, T, 1.f / (float)T)] : 0.0;
  }
  __syncthreads();
  for (; l0 < lines; l0 += stride) {
    double c[R + 1], sn[R], sq = (double)e0 * (double)e0;
#pragma unroll
    for (int f = 0; f <= R; ++f) c[f] = (double)e0;
#pragma unroll
    for (int f = 0; f < R; ++f) sn[f] = 0.0;
    seek(l0 + stride);
    e0 = element(0, true);
    int zero = 0;
    asm volatile("" : "+s"(zero));  // (the factors are read for each line: they are more than the registers)
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const double x = (double)a[u], y = (double)b[u], p = x + y, m = x - y;
      ask(u);
      sq = fma(x, x, fma(y, y, sq));
      const double *w = op + zero + u * K;
#pragma unroll
      for (int f = 0; f <= R; ++f) c[f] = fma(p, w[f], c[f]);
#pragma unroll
      for (int f = 0; f < R; ++f) sn[f] = fma(m, w[R + 1 + f], sn[f]);
      if (u % 2) __builtin_amdgcn_sched_barrier(0);
    }
    double q = 0.0;  // (coefficients past the last are left out, not weighted with 0: they are infinite with an infinite element)
#pragma unroll
    for (int f = 0; f < R; ++f)
      if (f + 1 <= r) q = fma(c[f + 1], c[f + 1], fma(sn[f], sn[f], q));
    s_t += fma(c[0], c[0], 2.0 * q);
    s_in += sq;
  }
}

template <int M, int YT, int W, int R>  // tiles of y coefficients, tiles of y, whole sixteens of folded x (up to 16 elements more are its rest), t
__global__ __launch_bounds__(kEbcChThreads, W == 1 ? 4 : 2) void ebc_channel_kernel(
    const float *__restrict__ err, const float *__restrict__ dense, long long total, int C, int T, int Y, int X, int n_ch, int gt,
    double *__restrict__ partials) {
  extern __shared__ __align__(16) double ebc_lds[];
  __shared__ double red[kEbcChWaves][2];
  // sums over the workgroup in a fixed order, valid in thread 0
  auto block_sums = [&](double (&v)[2]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2; ++i) v[i] = ebc_wave_sum(v[i]);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
      for (int i = 0; i < 2; ++i) red[threadIdx.x >> 6][i] = v[i];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      v[i] = red[0][i];
#pragma unroll
      for (int w = 1; w < kEbcChWaves; ++w) v[i] += red[w][i];
    }
  };
  int blk = blockIdx.x;
  if (blk >= n_ch) {
    blk -= n_ch;
    double sums[2] = {0.0, 0.0};
    if (blk < gt) {
      ebc_lines_t<R, R == 5 ? 11 : 17>(err, (long long)C * Y * X, T, Y * X, blk, gt, ebc_lds, sums[0], sums[1]);
      block_sums(sums);
      if (threadIdx.x == 0) {
        partials[0 * kEbcPartials + blk] = sums[1];
        partials[1 * kEbcPartials + blk] = sums[0];
      }
    } else {
      blk -= gt;
      sums[0] = ebc_squares<kEbcChThreads>(dense, total, blk, (int)gridDim.x - n_ch - gt);
      block_sums(sums);
      if (threadIdx.x == 0) partials[4 * kEbcPartials + blk] = sums[0];
    }
    return;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l16 = lane & 15, g = lane >> 4;
  const int KY = ebc_coefs(Y), KT = ebc_coefs(T), rx = X / 4, n_cos = rx / 16 + 1, PX = n_cos + (rx + 15) / 16;
  const int units = (C + kNumXcd - 1) / kNumXcd * kNumXcd * PX;
  // operands of the table for each step and lane (in registers they took 20 to 60 others to scratch memory), coef[t][ky][16]
  constexpr int SX = 4 * W + 4, SY = 4 * M * YT, ST = R == 5 ? 6 : 9, PT = R == 5 ? 1 : 2;
  double *tab_t = ebc_lds, *tab_y = tab_t + 2 * T, *tab_x = tab_y + 2 * Y, *op_y = tab_x + 2 * X, *op_t = op_y + 64 * SY,
         *op_x = op_t + 64 * ST * PT, *coef = op_x + 64 * SX;
  // (the groups of 16 x coefficients of a channel go to one XCD)
  auto channel = [&](int u) -> int { return u / (kNumXcd * PX) * kNumXcd + u % kNumXcd; };
  // Folded elements j = 0 .. X / 2 of row l16 of y tile yt of plane (c, t): of every whole 16 those of 4 g .. 4 g + 3, of the rest g
  // and every fourth; e_j and e_(X-j).  Rows past the end are out of range for the descriptor and arrive as zeros; what is loaded for
  // an element past the last, and as the mirror image of one that has none, is not used.
  // (All steps are taken, of zeros where there are no elements: a branch a step kept the operands' reads behind it.)
  const int folded = X / 2 + 1;  // (16 W <= folded <= 16 W + 16: see ebc_one_launch)
  const uint32_t plane = (uint32_t)(Y * X) * 4u;
  constexpr uint32_t kNowhere = 0x7fff0000u;
  struct Fold {
    float at[SX], mirror[SX];
  };
  auto load = [&](Fold &v, int c, int t, int yt) __attribute__((always_inline)) {
    typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
    const int y = 16 * yt + l16;
    const bool ok = c < C && t < T;  // uniform
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(err) + (long long)(ok ? c : 0) * T * Y * X + (long long)(ok ? t : 0) * Y * X, 0, ok ? (int)plane : 0, 0x00020000);
    const uint32_t row = y < Y ? (uint32_t)(y * X) * 4u : kNowhere;
    // (the mirror image of j = 0 would be the element behind the row: those of 1 to 3 are loaded with the one before them)
    const uint32_t ahead = row + 16u * g, back = row + 4u * (X - 3) - 16u * g, single = row + 4u * (16 * W + g),
                   single_back = row + 4u * (X - 16 * W - g);
#pragma unroll
    for (int u = 0; u < W; ++u) {
      const bool first = u == 0 && g == 0;
      const u32x4 q = __builtin_amdgcn_raw_buffer_load_b128(rs, ahead + 64u * u, 0, 0);
      const u32x4 m = __builtin_amdgcn_raw_buffer_load_b128(rs, back - 64u * u - (first ? 4u : 0u), 0, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        v.at[4 * u + i] = __uint_as_float(q[i]);
        v.mirror[4 * u + i] = __uint_as_float(m[3 - i]);  // (e_(X-j), in the first lanes that of j + 1: see mirror_of)
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v.at[4 * W + i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, single + 16u * i, 0, 0));
      v.mirror[4 * W + i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, single_back - 16u * i, 0, 0));
    }
  };
  // (at its use: a selection here would wait for the loads)
  auto mirror_of = [&](const Fold &v, int u) __attribute__((always_inline)) -> float {
    return u > 0 && u < 4 && g == 0 ? v.mirror[u > 0 ? u - 1 : 0] : v.mirror[u];
  };
  Fold even, odd;
  load(even, channel(blk), wave, 0);
  // (tables as ebc_table's)
  const float rt = 1.f / (float)T, ry = 1.f / (float)Y, rx1 = 1.f / (float)X;
  for (int m = threadIdx.x; m < T + Y + X; m += kEbcChThreads) {
    const int n = m < T ? T : m < T + Y ? Y : X, i = m < T ? m : m < T + Y ? m - T : m - T - Y;
    double *tab = m < T ? tab_t : m < T + Y ? tab_y : tab_x;
    double c, sn;
    sincospi(2.0 * (double)i / (double)n, &sn, &c);
    tab[i] = c;
    tab[n + i] = sn;
  }
  __syncthreads();
  // place of coefficient k's value at element j in a table of n: 0 the mean, then cosine and sine of each frequency (those
  // past K are computed and dropped)
  auto place = [&](int k, int K, int n, float rn, int j) __attribute__((always_inline)) -> int {
    const int f = k < K ? (k + 1) >> 1 : 0;
    return ((k & 1) == 0 && k > 0 && k < K ? n : 0) + ebc_mod(f * j, n, rn);
  };
  for (int i = wave; i < SY; i += kEbcChWaves) op_y[64 * i + lane] = tab_y[place(16 * (i / (4 * YT)) + l16, KY, Y, ry, 4 * (i % (4 * YT)) + g)];
  for (int i = wave; i < ST * PT; i += kEbcChWaves) op_t[64 * i + lane] = tab_t[place(16 * (i / ST) + l16, KT, T, rt, 4 * (i % ST) + g)];
  double s_xy = 0.0, s_xyt = 0.0;
  for (int unit = blk; unit < units; unit += n_ch) {
    const int c = channel(unit), q = unit / kNumXcd % PX;
    if (c >= C) continue;  // uniform
    const bool sine = q >= n_cos;
    const int fx = sine ? 16 * (q - n_cos) + l16 + 1 : 16 * q + l16;  // this lane's frequency
    const bool in_x = fx <= rx;
    const double wx = fx > 0 ? 2.0 : 1.0, sign = sine ? -1.0 : 1.0;
    for (int i = wave; i < SX; i += kEbcChWaves) {
      const int j = i < 4 * W ? 16 * (i / 4) + 4 * g + i % 4 : 16 * W + 4 * (i - 4 * W) + g;
      op_x[64 * i + lane] = tab_x[(sine ? X : 0) + ebc_mod((in_x ? fx : 0) * j, X, rx1)];
    }
    __syncthreads();
    // (two sets of registers in turn: a copy of what has been asked for would wait for it)
    ebc_f64x4 acc2[M];
#pragma unroll
    for (int m = 0; m < M; ++m) acc2[m] = ebc_f64x4{0.0, 0.0, 0.0, 0.0};
    int t = wave, yt = 0;
    auto tile = [&](const Fold &v, Fold &nxt) __attribute__((always_inline)) {
      const bool same = yt + 1 < YT;
      const int t1 = same ? t : t + kEbcChWaves, yt1 = same ? yt + 1 : 0;
      load(nxt, c, t1, yt1);
      ebc_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
      double bx[SX], ay[M][4];  // (all read before the first is used)
#pragma unroll
      for (int u = 0; u < SX; ++u) bx[u] = op_x[64 * u + lane];
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) ay[m][r] = op_y[64 * ((m * YT + yt) * 4 + r) + lane];
      __builtin_amdgcn_sched_barrier(0);
      auto step = [&](int u, int j, bool there) __attribute__((always_inline)) {
        float at = there ? v.at[u] : 0.f, mirror = there && j > 0 && 2 * j != X ? mirror_of(v, u) : 0.f;
        asm volatile("" : "+v"(at), "+v"(mirror));  // (selections of 32 bits, not of 64)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fma(sign, (double)mirror, (double)at), bx[u], acc, 0, 0, 0);
      };
#pragma unroll
      for (int u = 0; u < W; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) step(4 * u + i, 16 * u + 4 * g + i, true);
#pragma unroll
      for (int i = 0; i < 4; ++i) step(4 * W + i, 16 * W + 4 * i + g, 16 * W + 4 * i + g < folded);
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int m = 0; m < M; ++m)
          acc2[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(ay[m][r], acc[r], acc2[m], 0, 0, 0);
      if (!same) {
        double s_plane = 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int ky = 16 * m + 4 * r + g;
            const double x = acc2[m][r];
            // (coefficients past the last are left out, not weighted with 0: they are infinite with an infinite element)
            if (ky < KY) {
              if (in_x) s_plane = fma((ky > 0 ? 2.0 : 1.0) * x, x, s_plane);
              coef[(t * KY + ky) * 16 + l16] = x;
            }
            acc2[m][r] = 0.0;
          }
        s_xy = fma(wx, s_plane, s_xy);
      }
      t = t1;
      yt = yt1;
    };
    while (t < T) {
      tile(even, odd);
      if (t < T) tile(odd, even);
    }
    load(even, channel(unit + n_ch), wave, 0);
    __syncthreads();
    // over t: a wavefront has a row of y coefficients at a time (KY is odd: the rows of two t lie in different halves of the banks)
    for (int ky = wave; ky < KY; ky += kEbcChWaves) {
      const double w = ky > 0 ? 2.0 * wx : wx;
      double b[ST];
#pragma unroll
      for (int i = 0; i < ST; ++i) b[i] = 4 * i + g < T ? coef[((4 * i + g) * KY + ky) * 16 + l16] : 0.0;
#pragma unroll
      for (int p = 0; p < PT; ++p) {
        ebc_f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int i = 0; i < ST; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(op_t[64 * (p * ST + i) + lane], b[i], acc, 0, 0, 0);
        double s_row = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int kt = 16 * p + 4 * r + g;
          const double v = acc[r];
          if (in_x && kt < KT) s_row = fma((kt > 0 ? 2.0 : 1.0) * v, v, s_row);
        }
        s_xyt = fma(w, s_row, s_xyt);
      }
    }
    __syncthreads();
  }
  double sums[2] = {s_xy, s_xyt};
  block_sums(sums);
  if (threadIdx.x == 0) {
    partials[2 * kEbcPartials + blk] = sums[0];
    partials[3 * kEbcPartials + blk] = sums[1];
  }
}

__global__ __launch_bounds__(kEbcThreads) void ebc_total_kernel(double *__restrict__ partials, EbcFinish f,
                                                                double *__restrict__ out) {
  ebc_total(partials, f, out);
}

// a kernel as a type
template <auto K>
struct EbcKernel {
  static constexpr auto k = K;
};

// the two coefficient arrays (neither larger than the tensor), the partial sums with the tickets
static size_t ebc_workspace_doubles(long long total, int T, int Y, int X) {
  return 2 * (size_t)total + (size_t)(T + Y + X) + kEbcSums * (size_t)kEbcPartials;
}

// groups of 16 x coefficients of one kind (ebc_channel_kernel): cosines of the frequencies 0 .. X / 4, sines of 1 .. X / 4
static int ebc_x_groups(int X) { return X / 4 / 16 + 1 + (X / 4 + 15) / 16; }

// Whether ebc_channel_kernel is the better one.  Whole call, two launches through memory -> one and the total, us, one tensor again and
// again (from HBM where that is another matter).  It holds 16 to 48 folded elements of x (at 95 x 48 x 35 142 of 144 KB of LDS) and y
// and t up to its operands' tiles; of these sizes
// - enough channels: 16 x 23 x 40 x 80 24.9 -> 30.1, 24 x 22 x 40 x 64 23.8 -> 31.9, 32 x 23 x 30 x 48 19.0 -> 21.1 against 48 x 22 x
//   24 x 53 20.9 -> 18.1, 64 x 22 x 47 x 72 47.9 -> 38.8;
// - all workgroups of planes at once, two a CU with x below 64, one above: 256 x 12 x 24 x 56 (512 of them) 34.8 -> 31.4, 64 x 33 x 28 x
//   67 (192) 41.5 -> 34.3; a second and third round of them 72 x 33 x 34 x 68 (288) 55.5 -> 69.6, 160 x 21 x 22 x 72 45.9 -> 52.9,
//   1024 x 28 x 2 x 68 69.7 -> 219;
// - and bytes enough for what a workgroup does one after another (two planes a wavefront from t = 9, three from 17), which steps that are
//   mostly padding (x of 32 to 43) lengthen: 48 x 21 x 6 x 32 14.3 -> 16.8, 24 x 23 x 6 x 76 17.3 -> 20.3, against 128 x 20 x 6 x 48
//   20.9 -> 15.9 and, eight planes, 64 x 2 x 6 x 66 17.3 -> 11.6.
// Never t of 24 to 32, which costs as much as 35 here and one tile of coefficients, not two, there (56 x 28 x 20 x 80 26.2 -> 33.4); from
// 33 with bytes enough, 64 x 35 x 45 x 76 70.0 -> 54.9, not 80 x 34 x 17 x 66 33.2 -> 36.2.
// More rounds where they are full and the planes tall: x of 50 to 63, two a CU, 300 x 21 x 28 x 52 54.5 -> 46.7, 1024 x 17 x 28 x 60
// 165 -> 132, not 300 x 17 x 2 x 32 19.7 -> 27.7; above, two full ones, 128 x 33 x 45 x 80 120.4 -> 104.8 (from HBM 120.4 -> 115.5), 128 x 20
// x 45 x 67 65.5 -> 50.3, 128 x 21 x 45 x 88 81.9 -> 70.6; not 112 x 17 x 34 x 72 (448 workgroups, 6 to 12 % slower), 128 x 33 x 32 x 72
// (+2 to +7 %), nor t of 17 to 23 with x of 68 to 80, a fourth group of coefficients for one to four of them (128 x 23 x 45 x 80
// 73.8 -> 73.1, from HBM 74.9 -> 82.8).
static bool ebc_one_launch(long long C, int T, int Y, int X) {
  const long long total = C * T * Y * X;  // (32-bit byte offsets)
  const bool narrow = X < 64;
  if (X < 32 || X > 95 || T > (narrow ? 23 : 35) || Y > (narrow ? 31 : kEbcPlaneY) || total > 0x3fffffff) return false;
  const int PX = ebc_x_groups(X), units = (int)((C + kNumXcd - 1) / kNumXcd) * kNumXcd * PX;
  if (C * PX < (Y < 32 ? 96 : 192)) return false;
  const long long chain = T <= 8 ? 0 : X < 36 ? 1000000 : 65000LL * (T - 8);
  if (narrow)
    return units <= 256   ? X >= 44 || total >= chain
           : units <= 512 ? X >= 44 && total >= 2 * chain
                          : X >= 50 && T > 16 && Y >= 16;
  if (units <= 256) return T < 24 ? total >= chain : T > 32 && total >= (X < 68 ? 3200000 : 4500000);
  return Y >= 32 && units >= (X < 68 ? 384 : 481) && units <= 512 &&
         (T < 24 ? T > 16 && (X < 68 || X > 80) : T > 32 && Y >= 44);
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
  if (ebc_one_launch(C, T, Y, X)) {
    const bool low = Y < 32, wide = X >= 64;  // (2 (Y / 4) + 1 coefficients, X / 2 + 1 folded elements)
    const int PX = ebc_x_groups(X);
    const int ch_steps = (wide ? 12 : 8) + (low ? 8 : 24) + (T < 24 ? 6 : 18);  // operands of the table (ebc_channel_kernel)
    const size_t ch_lds = sizeof(double) * std::max(2 * (size_t)(T + Y + X) + 64 * (size_t)ch_steps + (size_t)T * KY * 16,
                                                    2 * (size_t)T + (T < 24 ? 11 * 12 : 17 * 18));
    const int units = (int)((C + kNumXcd - 1) / kNumXcd) * kNumXcd * PX, n_ch = std::min(units, kEbcPartials);
    auto rounds = [](long long n, long long most) -> int {  // workgroups: the fewest equal rounds of no more than `most`
      const long long r = (n + most - 1) / most;
      return (int)((n + r - 1) / r);
    };
    const int gt = rounds((lt.lines + kEbcChThreads - 1) / kEbcChThreads, 160);
    const int gd = (int)std::min<long long>((total + 16 * kEbcChThreads - 1) / (16 * kEbcChThreads), 96);
    const EbcFinish f{{gt, gt, n_ch, n_ch, gd}, (double)T, (double)Y * X, {w[0], w[1], w[2], w[3]}, epsilon};
    auto run = [&](auto kern) -> int {
      static DeviceFlags attr_set;  // (per instantiation: the lambda's argument has a type of its own)
      const int dev = current_device();
      if (dev < 0) return fail(HEART_EHIP, "heart_ebc_band_error: cannot identify the current device");
      if (hipError_t e = set_max_lds_once(attr_set, dev, reinterpret_cast<const void *>(kern.k), kEbcChLds))
        return fail(HEART_EHIP, "hipFuncSetAttribute(band error LDS): %s", hipGetErrorString(e));
      hipLaunchKernelGGL(kern.k, dim3((unsigned)(n_ch + gt + gd)), dim3(kEbcChThreads), ch_lds, st, err, dense, total, (int)C, T, Y,
                         X, n_ch, gt, partials);
      return HEART_OK;
    };
    if (int rc = !wide    ? run(EbcKernel<ebc_channel_kernel<1, 2, 1, 5>>{})
                 : T < 24 ? (low ? run(EbcKernel<ebc_channel_kernel<1, 2, 2, 5>>{}) : run(EbcKernel<ebc_channel_kernel<2, 3, 2, 5>>{}))
                          : (low ? run(EbcKernel<ebc_channel_kernel<1, 2, 2, 8>>{}) : run(EbcKernel<ebc_channel_kernel<2, 3, 2, 8>>{})))
      return rc;
    hipLaunchKernelGGL(ebc_total_kernel, dim3(1), dim3(kEbcThreads), 0, st, partials, f, out);
    return check_launch("ebc kernels");
  }
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
