// heart_scores_antidiag: an antidiagonal-style block-importance estimator that feeds
// heart_mask_topp through its scores_in argument, as an alternative to the pooled scores.
// The paper leaves importance ranking to the sparse-attention backbone and names this
// family with its setting (antidiagonal scoring, stride 16, blocks of 128 tokens: appendix
// on baseline configurations); the definition implemented here is
//   S = stride, block = 8 S, tokens past N are zero vectors,
//   L[a,b]  = 1/(S sqrt(D)) * sum_{r<S} q[S a + S-1-r] . k[S b + r]   (the antidiagonal of
//             the S x S tile (a,b) of Q K^T), a, b < M = ceil(N/S)
//   P[a,:]  = softmax_b L[a,:]
//   score[I,J] = mean_{a in block I} sum_{b in block J} P[a,b]
//
// L is one bf16 GEMM per head: row a of the left operand is the S token rows of reduced
// query a in reverse order, S*D contiguous-by-row elements, row b of the right operand the
// S token rows of reduced key b in order.  2 M^2 S D FLOP per head on the matrix cores
// (v_mfma_f32_16x16x32_bf16), MFMA-bound, and bound by power while a full chip works: matrix instructions alone, operands N(0, 1) in
// registers, sustain 1710 to 1800 TFLOP/s as 32x32x16 and 2020 to 2190 as 16x16x32 (half as many accumulator reads and writes a
// FLOP), most where consecutive ones add to the same accumulator (one by one 2050, two 2165, four 2160).  With the same tiles and the
// same operand reads estimator and selection of 40 heads of 32760 tokens take 645 us with 32x32x16 and 613 with this (the same bits;
// under counters the tile kernel has 1.10 million active cycles at 1.85 GHz and 1.16 at 2.02).
//
// Kernel 1 (antidiag_tile): one workgroup (8 wavefronts) per 256 x 256 tile of L (128 FLOP
//   per operand byte, which keeps the operand stream from L2 below what it delivers), or (4) per 128 x 128.  The
//   contraction runs in stages of 64 elements (half a token row at D = 128): both operand
//   tiles go from global memory straight into LDS (`buffer_load ... lds`, 16-byte chunks
//   XOR-swizzled by row so that the fragment reads are conflict free), double-buffered
//   (128 KB, 64 KB; 128 KB in four buffers for one small tile a CU), one barrier per stage, the loads of the next
//   stage in flight during the MFMAs of the current one (lines of later stages requested into the L2 as well: 613 ->
//   625 us); fragments are read two key tiles ahead, and fragment reads and loads are issued between the MFMAs, one or two
//   behind each: all eight loads of a wavefront in one go, right after the barrier, held the MFMAs behind them
//   back until the address unit had taken them (estimator and selection, 40 heads of 32760 tokens 674 -> 656 us,
//   10 of 75600 960 -> 917, 20 of 32760 at D = 64 200 -> 184, 12 of 20280 in blocks of 64 193 -> 180, six of 3565
//   29.3 -> 26.8).  With a full chip the flight time of the loads does not count: stages of half the depth, five
//   buffers and four stages ahead took 709 to 720 us in the place of 660, four wavefronts of 128 x 128, one a SIMD,
//   730.  A wavefront owns 64 (32) reduced queries against 128 reduced keys (S^T layout: keys
//   along the accumulator rows), so a query's maximum over those keys is a per-lane
//   reduction plus two exchanges among the four lanes that share the query (one between two, in the small tiles).  The epilogue writes one record per
//   (reduced query, 128 keys): the maximum m and the 16 sums over 8 keys of exp2(L - m).
//   Tiles are independent.
// Kernel 2 (antidiag_combine): one workgroup per query block: global maximum and
//   normaliser of each of its reduced queries from the records, then the mean over the
//   reduced queries of the rescaled key-block sums.
#include "heart_internal.h"

namespace heart {

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t ad_u32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 ad_bf16x8;
typedef __attribute__((ext_vector_type(4))) float ad_f32x4;
typedef __attribute__((ext_vector_type(16))) float ad_f32x16;
union AdFrag {
  ad_u32x4 u;
  ad_bf16x8 v;
};

constexpr int kAdTile = 256;                     // reduced rows per tile side (or half as many: launch_antidiag)
constexpr int kAdRowB = 128;                     // bytes per tile row and stage (64 bf16)
constexpr int kAdKeysPerBlock = 8;               // reduced keys per key block (block = 8 S)
constexpr float kAdFused = 1048576.f;             // largest logit (log2 units) that is scaled and subtracted in one operation
constexpr int kAdLookHeads = 256;                // most heads whose refresh flags every workgroup looks at
constexpr int ad_lds(int tile, int bufs) { return 2 * bufs * tile * kAdRowB; }  // stages x two operands (128 KB, 64 KB)

// raw buffer descriptor (base, size in bytes) as four words in scalar registers, for the
// hand-written LDS-direct loads; accesses past `bytes` return zeros
__device__ __forceinline__ ad_u32x4 ad_rsrc_words(const uint16_t *base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  ad_u32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
  r.z = __builtin_amdgcn_readfirstlane(bytes);
  r.w = 0x00020000u;
  return r;
}

}  // namespace

// kTile = 256: 8 wavefronts of 64 queries x 128 keys; 128: 4 of 32 queries x 128 keys, two workgroups a CU (kBufs stage buffers; 4: one)
template <int D, int kTile, int kBufs>
__global__ __launch_bounds__(2 * kTile, 2) void antidiag_tile_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k, long long qsb, long long qsh,
    long long qsn, long long ksb, long long ksh, long long ksn, int H, int BH, int N, int S, int M,
    int MTQ, int MT, float scale_log2, const unsigned char *__restrict__ refresh, float *__restrict__ esum,
    float *__restrict__ mref) {
  extern __shared__ __align__(1024) unsigned char smem[];
  constexpr int kAdTileB = kTile * kAdRowB;  // bytes of one operand tile of one stage
  const int t = threadIdx.x;
  const int lane = t & 63;
  // workgroup -> (head, tile): workgroup ids are dealt round-robin to the 8 XCDs; an XCD takes a contiguous
  // eighth of the tiles of the refreshed heads, head by head, so that a head's operand rows are shared
  // through one L2 or a few, and no XCD has more to do than another (before, whole heads went to the XCDs in turn: 12
  // heads of 64 tiles 232 -> 179 us, one head 99 -> 47).  With hundreds of heads a look at all flags costs more than
  // the tiles of reused heads, which end at once.
  const int tiles_k = MT / (kTile / 128);  // (every record of 128 keys is written, also past the end)
  const unsigned tph = (unsigned)(MTQ * tiles_k), x = blockIdx.x % kNumXcd;
  const bool look = refresh && BH <= kAdLookHeads;
  unsigned long long set[kAdLookHeads / 64];  // refreshed heads
  unsigned n_heads = (unsigned)BH;
  if (look) {
    unsigned char f[kAdLookHeads / 64];
#pragma unroll
    for (int c = 0; c < kAdLookHeads / 64; ++c) f[c] = refresh[min(64 * c + lane, BH - 1)];
    n_heads = 0;
#pragma unroll
    for (int c = 0; c < kAdLookHeads / 64; ++c) {
      set[c] = __ballot(64 * c + lane < BH && f[c] != 0);
      n_heads += (unsigned)__popcll(set[c]);
    }
  }
  const unsigned long long items = (unsigned long long)n_heads * tph;
  const unsigned w = (unsigned)(items * x / kNumXcd) + blockIdx.x / kNumXcd;
  if (w >= (unsigned)(items * (x + 1) / kNumXcd)) return;
  int bh = (int)(w / tph);
  const int tile = (int)(w - (unsigned)bh * tph);
  if (look) {
    int rank = bh;
#pragma unroll
    for (int c = 0; c < kAdLookHeads / 64; ++c) {
      const int n = __popcll(set[c]);
      const bool mine = ((set[c] >> lane) & 1) && __popcll(set[c] & ((1ull << lane) - 1ull)) == rank;
      const unsigned long long m = __ballot(mine);
      if (rank >= 0 && rank < n) bh = 64 * c + __ffsll((long long)m) - 1;
      rank -= n;  // (negative once found)
    }
  } else if (refresh && !refresh[bh]) {
    return;  // reused head: its cached mask persists, no scores needed
  }
  const int tq = tile / tiles_k, tk = tile % tiles_k;
  const int b = bh / H, h = bh % H;

  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wi = wave >> 2;  // which 128 keys of the tile
  const int wj = wave & 3;   // which quarter of the tile's queries

  const ad_u32x4 q_rs = ad_rsrc_words(q + b * qsb + h * qsh, (uint32_t)((long long)N * qsn * 2));
  const ad_u32x4 k_rs = ad_rsrc_words(k + b * ksb + h * ksh, (uint32_t)((long long)N * ksn * 2));
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem;

  // Staging by LDS-direct loads: one instruction moves 16 bytes per lane to 1 KB of consecutive
  // LDS, i.e. 8 tile rows; lane l lands at chunk position l % 8 of row l / 8 and therefore
  // fetches the global chunk (l % 8) ^ f(row) (the XOR swizzle is applied on the global side).
  // Wavefront w issues instructions 4 w .. 4 w + 3 of each operand tile.  The whole byte
  // offset goes through the vector offset, which the descriptor range-checks: rows of tokens
  // >= N are out of range and arrive as zeros.
  constexpr int SPR = D / 64;  // stages per token row
  uint32_t q_dma[4], k_dma[4];
  {
    const int drow = lane >> 3, dp = lane & 7;
#pragma unroll
    for (int ii = 0; ii < 4; ++ii) {
      const int row = 8 * (4 * wave + ii) + drow;
      const uint32_t chunk = (uint32_t)(dp ^ ((row >> 1) & 7));
      // (token index of sub-row 0; the stage adds its sub-row)
      q_dma[ii] = (uint32_t)(S * (kTile * tq + row)) * (uint32_t)(qsn * 2) + chunk * 16u;
      k_dma[ii] = (uint32_t)(S * (kTile * tk + row)) * (uint32_t)(ksn * 2) + chunk * 16u;
    }
  }
  // (the compiler does not see the LDS write of these instructions: their completion is
  // awaited explicitly before the barrier that publishes the stage)
  constexpr int kLoads = 8;  // of a stage and wavefront: the keys' and the queries' in turn
  auto dma = [&](int st, int buf, int i) __attribute__((always_inline)) {
    const int r = st / SPR, d0 = (st % SPR) * 64, ii = i >> 1;
    const uint32_t dst = smem_lds + (uint32_t)((buf * 2 + (i & 1)) * kAdTileB + (4 * wave + ii) * 1024);
    uint32_t m0_saved;  // (M0 carries the LDS destination; saved and restored for the compiler)
    if (i & 1) {
      const uint32_t qo = (uint32_t)(S - 1 - r) * (uint32_t)(qsn * 2) + (uint32_t)d0 * 2u;
      asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                   : "=&s"(m0_saved) : "s"(dst), "v"(q_dma[ii] + qo), "s"(q_rs) : "memory");
    } else {
      const uint32_t ko = (uint32_t)r * (uint32_t)(ksn * 2) + (uint32_t)d0 * 2u;
      asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                   : "=&s"(m0_saved) : "s"(dst), "v"(k_dma[ii] + ko), "s"(k_rs) : "memory");
    }
  };
  auto wait_loads_and_barrier = [&]() __attribute__((always_inline)) {
    // (the loads of the next stage; those of the stages behind it may be in flight)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kBufs - 2) * kLoads) : "memory");
    __syncthreads();
  };
  // Per stage: the barrier that hands over the next stage sits before the MFMAs of the stage's last quarter.  By then a
  // wavefront has completed all its reads of the current buffer and its loads of the next stage into the other one;
  // behind those MFMAs it issues the first half of the loads of the stage kBufs on into the buffer just released, behind
  // those of the next quarter the other half (the later a load, the shorter its flight: all within the
  // first quarter, or three, 0.5 to 2 % slower).  Loads past the last stage repeat the last stage (into a buffer
  // nobody reads any more).
  const int n_stages = kTile * tk < M ? S * SPR : 0;  // (a tile of keys past the end: records without weight)
  const int last = max(n_stages - 1, 0);
  constexpr int kHalf = kLoads / 2;
#pragma unroll
  for (int st = 0; st < kBufs - 1; ++st)
#pragma unroll
    for (int i = 0; i < kLoads; ++i) dma(min(st, last), st, i);
  wait_loads_and_barrier();
#pragma unroll
  for (int i = 0; i < kHalf; ++i) dma(min(kBufs - 1, last), kBufs - 1, i);
  auto no_extra = [](int) {};
  // ---- epilogue: record of (reduced query, 128 keys): maximum and 16 key-block sums ----------
  const float ninf = -__builtin_inff();
  const int key0 = kTile * tk + 128 * wi;
  const int rec = kTile / 128 * tk + wi;  // index of the 128-key record
  const int NbP = 16 * MT;

  if constexpr (kTile == 256) {
    constexpr int QT = 4, KT = 8;  // tiles of 16: of the queries, of the keys
    const int l16 = lane & 15, grp = lane >> 4;
    // fragment of contraction step ks (32 elements) of tile row 16 x + l16: chunk 4 ks + grp
    uint32_t foff[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) foff[ks] = (uint32_t)(l16 * kAdRowB + (((4 * ks + grp) ^ ((l16 >> 1) & 7)) * 16));

    ad_f32x4 acc[KT][QT];
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt) acc[kt][qt] = ad_f32x4{0.f, 0.f, 0.f, 0.f};

    // Fragments: of the queries (B operand) those of a whole stage, of the keys (A operand) those of two key tiles and, arriving, of
    // the next two.  A pair of key tiles is worked on query tile by query tile, both contraction steps of an accumulator after one
    // another (two MFMAs in a row on one accumulator take less power than on two).  Behind the last pair of a stage, each when its
    // last MFMA has been issued, the queries of the next stage are read.
    AdFrag fb[QT][2], fa[2][2][2];  // [tile][step], [pair][tile][step]
    constexpr int kMfmas = 4 * QT;  // of a pair of key tiles
    auto read_a = [&](int buf, int pair, int i) __attribute__((always_inline)) {  // i: tile and step
      const unsigned char *A = smem + buf * 2 * kAdTileB + wi * 128 * kAdRowB;
      fa[pair & 1][i >> 1][i & 1].u = *reinterpret_cast<const ad_u32x4 *>(A + (2 * pair + (i >> 1)) * 16 * kAdRowB + foff[i & 1]);
    };
    auto read_b = [&](int buf, int qt, int ks) __attribute__((always_inline)) {
      const unsigned char *B = smem + buf * 2 * kAdTileB + kAdTileB + wj * 16 * QT * kAdRowB;
      fb[qt][ks].u = *reinterpret_cast<const ad_u32x4 *>(B + qt * 16 * kAdRowB + foff[ks]);
    };
    // The MFMAs of one pair of key tiles; behind the i-th what extra(i) issues, behind the first ones the reads of the next pair's
    // fragments (of buffer `buf`).
    auto pair_step = [&](int pair, int buf, auto &&extra) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < kMfmas; ++i) {
        const int qt = i >> 2, kt = (i >> 1) & 1, ks = i & 1;
        acc[2 * pair + kt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[pair & 1][kt][ks].v, fb[qt][ks].v,
                                                                         acc[2 * pair + kt][qt], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (j * (kMfmas / 2) / 4 == i) read_a(buf, (pair + 1) & 3, j);
        extra(i);
        __builtin_amdgcn_sched_barrier(0);
      }
    };

#pragma unroll
    for (int j = 0; j < 4; ++j) read_a(0, 0, j);
#pragma unroll
    for (int j = 0; j < 2 * QT; ++j) read_b(0, j >> 1, j & 1);
    for (int st = 0; st < n_stages; ++st) {
      const int buf = st % kBufs, buf1 = (st + 1) % kBufs, bufp = (st + kBufs - 1) % kBufs;
      const int st1 = min(st + kBufs - 1, last), st2 = min(st + kBufs, last);
      pair_step(0, buf, [&](int i) {
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
          if (j * kMfmas / kHalf == i) dma(st1, bufp, kHalf + j);
      });
      pair_step(1, buf, no_extra);
      pair_step(2, buf, no_extra);
      wait_loads_and_barrier();
      __builtin_amdgcn_sched_barrier(0);
      pair_step(3, buf1, [&](int i) {
        if ((i & 2) != 0) read_b(buf1, i >> 2, i & 1);  // (tile i / 4 has no MFMA after this one that reads step i % 2)
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
          if (j * kMfmas / kHalf == i) dma(st2, buf, j);
      });
    }
    // loads of the repeated last stage may still be in flight towards LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // accumulator element r of key tile kt: reduced key key0 + 16 kt + 4 grp + r
#pragma unroll
    for (int qt = 0; qt < QT; ++qt) {
      if (key0 + 128 > M) {  // (uniform: the records of the last keys)
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (key0 + 16 * kt + 4 * grp + r >= M) acc[kt][qt][r] = ninf;
      }
      // The maximum of the logits as they come out of the matrix cores, and exp2(scale L - scale max) in one fused
      // operation each (one rounding less than scaled logits and their difference, and two instructions).
      float m = ninf;
#pragma unroll
      for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r) m = fmaxf(m, acc[kt][qt][r]);
      {
        uint32_t s0, s1;
        swap_rows16(__float_as_uint(m), s0, s1);
        m = fmaxf(__uint_as_float(s0), __uint_as_float(s1));
        swap_halves32(__float_as_uint(m), s0, s1);
        m = fmaxf(__uint_as_float(s0), __uint_as_float(s1)) * scale_log2;
      }
      // The fused operation keeps what `m` was rounded by (up to 2^-24 of it), and from |m| = 2^31 on its exponential leaves
      // fp32: logits that large are scaled and rounded first, so that the largest is exactly its own reference.  (No time: estimator and
      // selection of 40 heads of 256 blocks 620.5 and 620.6 us.)
      float scale = scale_log2;
      if (__any(fabsf(m) > kAdFused)) {
        scale = 1.f;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) acc[kt][qt] *= scale_log2;
      }
      // (a record whose 128 keys are all past the end has m = -inf and all sums zero)
      const float mm = m == ninf ? 0.f : m;
      // Sums over the 8 keys of a key block: two lane groups hold four each (block 2 kt: groups 0 and 1).  z[p], of the key tiles
      // 2 p and 2 p + 1, has the sums of the blocks 4 p + 0, 2, 1, 3 in the groups 0 to 3; transposed, group g has blocks 4 g ..
      uint32_t z[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float s[2] = {0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[j] += __builtin_amdgcn_exp2f(fmaf(acc[2 * p + j][qt][i], scale, -mm));
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(s[0]), __float_as_uint(s[1]), false, false);
        z[p] = __float_as_uint(__uint_as_float(r[0]) + __uint_as_float(r[1]));
      }
      const auto h0 = __builtin_amdgcn_permlane32_swap(z[0], z[2], false, false);
      const auto h1 = __builtin_amdgcn_permlane32_swap(z[1], z[3], false, false);
      const auto v0 = __builtin_amdgcn_permlane16_swap(h0[0], h1[0], false, false);
      const auto v1 = __builtin_amdgcn_permlane16_swap(h0[1], h1[1], false, false);
      const int a = kTile * tq + 16 * QT * wj + 16 * qt + l16;
      if (a < M) {
        float *dst = esum + ((size_t)bh * M + a) * NbP + 16 * rec + 4 * grp;
        *reinterpret_cast<float4 *>(dst) = make_float4(__uint_as_float(v0[0]), __uint_as_float(v1[0]),
                                                       __uint_as_float(v0[1]), __uint_as_float(v1[1]));
        if (grp == 0) mref[((size_t)bh * M + a) * MT + rec] = m;
      }
    }
  } else {
    // (the same in tiles of 32: with few tiles power is not what counts, and reads and small MFMAs get in each other's way: six heads of
    // 5000 tokens 25.5 us, 26.6 with the tiles of 16; 24 heads of 6400 37.3, 40.0.  In large tiles, which short launches take too, that
    // is next to nothing: tile kernel and combine with the tiles of 16 in place of these, one round of 144 to 256 workgroups 23.0 ->
    // 23.3, 57.9 -> 58.1, 69.4 -> 69.4, 67.4 -> 66.3, 61.8 -> 57.6 us, two 60 of nine 137.2 -> 139.1, 8 of 64 124.1 -> 123.2, half the depth
    // 69.5 -> 65.5, ten 612 -> 595: from 2 % more to 7 % less, and the more tiles a head has the less)
    const int l32 = lane & 31, hf = lane >> 5;
    // fragment of contraction step ks (16 elements) of tile row 32 x + l32: chunk 2 ks + hf
    uint32_t foff[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) foff[ks] = (uint32_t)(l32 * kAdRowB + (((2 * ks + hf) ^ ((l32 >> 1) & 7)) * 16));

    ad_f32x16 acc[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[kt][r] = 0.f;

    // the fragments of one contraction step: 4 of the keys (A operand), one of the queries
    struct Frags {
      AdFrag a[4], b;
    };
    constexpr int kFrags = 5, kMfmas = 4;
    auto read_frag = [&](Frags &f, int buf, int ks, int i) __attribute__((always_inline)) {
      const unsigned char *A = smem + buf * 2 * kAdTileB + wi * 128 * kAdRowB;
      const unsigned char *B = smem + buf * 2 * kAdTileB + kAdTileB + wj * 32 * kAdRowB;
      if (i == 0)
        f.b.u = *reinterpret_cast<const ad_u32x4 *>(B + foff[ks]);
      else
        f.a[i - 1].u = *reinterpret_cast<const ad_u32x4 *>(A + (i - 1) * 32 * kAdRowB + foff[ks]);
    };
    // The MFMAs of one contraction step; behind those of the first half the reads of the next step's fragments (step ks of
    // buffer `buf`), behind each what extra(i) issues.
    auto step = [&](const Frags &f, Frags &next, int buf, int ks, auto &&extra) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < kMfmas; ++i) {
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.a[i].v, f.b.v, acc[i], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < kFrags; ++j)
          if (j * (kMfmas / 2) / kFrags == i) read_frag(next, buf, ks, j);
        extra(i);
        __builtin_amdgcn_sched_barrier(0);
      }
    };

    Frags f0, f1;
#pragma unroll
    for (int j = 0; j < kFrags; ++j) read_frag(f0, 0, 0, j);
    for (int st = 0; st < n_stages; ++st) {
      const int buf = st % kBufs, buf1 = (st + 1) % kBufs, bufp = (st + kBufs - 1) % kBufs;
      const int st1 = min(st + kBufs - 1, last), st2 = min(st + kBufs, last);
      step(f0, f1, buf, 1, [&](int i) {
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
          if (j * kMfmas / kHalf == i) dma(st1, bufp, kHalf + j);
      });
      step(f1, f0, buf, 2, no_extra);
      step(f0, f1, buf, 3, no_extra);
      wait_loads_and_barrier();
      __builtin_amdgcn_sched_barrier(0);
      step(f1, f0, buf1, 0, [&](int i) {
#pragma unroll
        for (int j = 0; j < kHalf; ++j)
          if (j * kMfmas / kHalf == i) dma(st2, buf, j);
      });
    }
    // loads of the repeated last stage may still be in flight towards LDS
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // accumulator element r of key tile kt: reduced key key0 + 32 kt + 8 (r / 4) + 4 hf + r % 4
    if (key0 + 128 > M) {  // (uniform: the records of the last keys)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (key0 + 32 * kt + 8 * (r >> 2) + 4 * hf + (r & 3) >= M) acc[kt][r] = ninf;
    }
    float m = ninf;
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int r = 0; r < 16; ++r) m = fmaxf(m, acc[kt][r]);
    {
      uint32_t s0, s1;
      swap_halves32(__float_as_uint(m), s0, s1);
      m = fmaxf(__uint_as_float(s0), __uint_as_float(s1)) * scale_log2;
    }
    float scale = scale_log2;
    if (__any(fabsf(m) > kAdFused)) {
      scale = 1.f;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[kt][r] *= scale_log2;
    }
    const float mm = m == ninf ? 0.f : m;
    float sums[4][4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) s += __builtin_amdgcn_exp2f(fmaf(acc[kt][4 * g + i], scale, -mm));
        uint32_t s0, s1;
        swap_halves32(__float_as_uint(s), s0, s1);
        sums[kt][g] = __uint_as_float(s0) + __uint_as_float(s1);
      }
    const int a = kTile * tq + 32 * wj + l32;
    if (a < M) {
      float *dst = esum + ((size_t)bh * M + a) * NbP + 16 * rec + 8 * hf;
      // lower-half lanes write key blocks 0..7 of the record, upper-half lanes 8..15
      *reinterpret_cast<float4 *>(dst) = hf ? make_float4(sums[2][0], sums[2][1], sums[2][2], sums[2][3])
                                            : make_float4(sums[0][0], sums[0][1], sums[0][2], sums[0][3]);
      *reinterpret_cast<float4 *>(dst + 4) = hf ? make_float4(sums[3][0], sums[3][1], sums[3][2], sums[3][3])
                                                : make_float4(sums[1][0], sums[1][1], sums[1][2], sums[1][3]);
      if (hf == 0) mref[((size_t)bh * M + a) * MT + rec] = m;
    }
  }
}

// One workgroup (4 wavefronts) per (head, query block).  A wavefront normalises two of the
// block's 8 reduced queries on its own (global maximum over the records, normaliser, both
// wave-wide reductions; the loads of both rows are issued before either is reduced), leaves
// the normalised key-block masses in LDS, and after one barrier the workgroup averages the
// 8 rows.  A lane has four key blocks at a time (one load; they share a record, whose maximum is one more), JQ times: 16 MT <=
// 256 JQ.  Bound by the records' bytes at many heads, by latency at few (estimator and selection with one key block a load -> four:
// 40 heads of 256 blocks 627 -> 619 us; eight heads of 13230 tokens at D = 64, inputs from HBM, 33.9 -> 33.1, six of 5250 27.6 -> 27.1).
template <int JQ>
__global__ __launch_bounds__(256) void antidiag_combine_kernel(int Nb, int M, int MT,
                                                              const unsigned char *__restrict__ refresh,
                                                              const float *__restrict__ esum,
                                                              const float *__restrict__ mref,
                                                              float *__restrict__ scores) {
  constexpr int RQ = kAdKeysPerBlock;       // reduced queries per query block
  extern __shared__ __align__(16) float s_w[];  // [RQ][NbP]
  const int I = blockIdx.x % Nb;
  const long long bh = blockIdx.x / Nb;
  if (refresh && !refresh[bh]) return;
  const int NbP = 16 * MT;
  const int a0 = I * RQ;
  const int na = min(RQ, M - a0);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  float mr[2], mj[2][JQ];
  float4 w[2][JQ];
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int rr = wave + 4 * x;
    const size_t row = (size_t)bh * M + a0 + (rr < na ? rr : 0);  // (rows past the end: loads of row 0, unused)
    mr[x] = lane < MT ? mref[row * MT + lane] : -__builtin_inff();
#pragma unroll
    for (int u = 0; u < JQ; ++u) {
      const int J = 4 * (lane + 64 * u);
      w[x][u] = J < NbP ? *reinterpret_cast<const float4 *>(esum + row * NbP + J) : make_float4(0.f, 0.f, 0.f, 0.f);
      mj[x][u] = J < NbP ? mref[row * MT + (J >> 4)] : 0.f;
    }
  }
#pragma unroll
  for (int x = 0; x < 2; ++x) {
    const int rr = wave + 4 * x;
    const float m = wave_max_f32(mr[x]);
    float part = 0.f;
#pragma unroll
    for (int u = 0; u < JQ; ++u) {
      const float f = 4 * (lane + 64 * u) < NbP ? __builtin_amdgcn_exp2f(mj[x][u] - m) : 0.f;
      w[x][u] = make_float4(w[x][u].x * f, w[x][u].y * f, w[x][u].z * f, w[x][u].w * f);
      part += (w[x][u].x + w[x][u].y) + (w[x][u].z + w[x][u].w);
    }
    const float inv = rr < na ? 1.f / wave_sum_f32(part) : 0.f;
#pragma unroll
    for (int u = 0; u < JQ; ++u) {
      const int J = 4 * (lane + 64 * u);
      if (J < NbP)
        *reinterpret_cast<float4 *>(s_w + rr * NbP + J) =
            make_float4(w[x][u].x * inv, w[x][u].y * inv, w[x][u].z * inv, w[x][u].w * inv);
    }
  }
  __syncthreads();
  const float inv_na = 1.f / (float)na;
  for (int J = t; J < Nb; J += 256) {
    float s = 0.f;
#pragma unroll
    for (int rr = 0; rr < RQ; ++rr) s += s_w[rr * NbP + J];
    scores[((size_t)bh * Nb + I) * Nb + J] = s * inv_na;
  }
}

size_t antidiag_workspace_bytes(const heart_shape &s, int stride) {
  const size_t M = ((size_t)s.N + stride - 1) / stride;
  const size_t MT = 2 * ((M + kAdTile - 1) / kAdTile);  // records of 128 keys per reduced query
  return (size_t)s.B * s.H * M * (16 * MT + MT) * sizeof(float);
}

int launch_antidiag(const heart_shape &s, const void *q, const void *k, int stride,
                    const unsigned char *refresh, float *scores, float *workspace, hipStream_t st) {
  const int S = stride;
  const int M = (s.N + S - 1) / S;
  const int MT2 = (M + kAdTile - 1) / kAdTile;
  const int MT = 2 * MT2;
  const int Nb = (s.N + s.block - 1) / s.block;
  const int BH = s.B * s.H;
  if (MT > 64)  // one wavefront reads a reduced query's records in the combine kernel
    return fail(HEART_EUNSUPPORTED, "heart_scores_antidiag: more than 8192 reduced rows");
  // the kernel addresses one head's rows through 32-bit buffer offsets, up to the end of
  // the last tile
  const long long rows = (long long)S * kAdTile * MT2 + S;
  if (rows * s.q_stride[2] * 2 > 0xffffffffLL || rows * s.k_stride[2] * 2 > 0xffffffffLL)
    return fail(HEART_EUNSUPPORTED,
                "heart_scores_antidiag: (N + 257 * stride) * token stride * 2 bytes must stay below 4 GiB");
  const int dev = current_device();
  if (dev < 0) return fail(HEART_EHIP, "heart_scores_antidiag: cannot identify the current device");
  // Tiles of 128 x 128, two workgroups a CU, where they fill the chip better: a round of them takes 0.5 to 0.6 of the
  // time of a round of 256 x 256, which move half the operand bytes per FLOP but come one to a CU.  Measured (tile and
  // combine kernel, 256 -> 128, heads of tiles of 32 stages: D = 128, stride 16): 13 heads of one tile 44.8 -> 20.5 us, one head of 64
  // tiles 45.2 -> 24.1, 13 of nine 45.5 -> 38.0; 20 of nine 62.9 -> 77.0, 12 of 64 184 -> 229, 40 of 64 595 -> 763.  (The same bits.)  Three
  // rounds in the place of two are 0.92 to 1.08 times as fast with 32 stages (8 of 36 99.1 -> 106.6, 30 of nine 107.5 -> 114.9, 24 of 16
  // 120.6 -> 120.8, 31 of nine 113.2 -> 109.6, 300 of one 168.8 -> 156.8), 0.98 to 1.08 with 16 (10 of 36 59.1 -> 60.4, 30 of nine 59.0 ->
  // 59.6, 8 of 36 57.1 -> 53.6, 300 of one 97.1 -> 90.4), 1.01 to 1.14 with 8; four of three 0.96 to 1.09 (57 of nine 131.3 -> 137.0, 33 of 16
  // 146.4 -> 138.3), 1.00 to 1.12 with 16.
  const int n_cu = cu_count(dev);
  if (n_cu <= 0) return fail(HEART_EHIP, "heart_scores_antidiag: cannot query the number of CUs");
  // Only the device knows how many heads `refresh` names, so small tiles then have to be the better ones for any number of
  // them, that is for the most heads of every number of rounds of large ones (30 heads of nine tiles, of which 16 refresh: 59
  // us, 73 with small tiles, at half the depth better for all 30 or as good).
  const long long large_h = (long long)MT2 * MT2, small_h = (long long)((M + 127) / 128) * MT;  // tiles of a head
  auto rounds = [](long long n, long long places) { return (n + places - 1) / places; };
  bool few = true;
  for (long long r = refresh ? rounds(large_h, n_cu) : rounds(BH * large_h, n_cu), heads = 0; few && heads < BH; ++r) {
    heads = refresh ? std::min<long long>(BH, r * n_cu / large_h) : BH;
    few = 10 * rounds(heads * small_h, 2 * n_cu) < (s.D * S >= 2048 ? 15 : 16) * r;
  }
  const int tile = few ? kAdTile / 2 : kAdTile, MTQ = (M + tile - 1) / tile;
  const long long grid = ((long long)BH * MTQ * (few ? MT : MT2) + kNumXcd - 1) / kNumXcd * kNumXcd;
  if (grid > 0x7fffffffLL || (long long)BH * Nb > 0x7fffffffLL)
    return fail(HEART_EUNSUPPORTED, "heart_scores_antidiag: grid too large");
  // One small tile a CU: four buffers, since nothing else is there to cover the flight of the loads
  // (estimator and selection, inputs from HBM, two buffers -> four: six heads of 5250 tokens 41.4 -> 27.6 us, 13 of 1590 33.3 -> 26.4;
  // inputs in the caches 31.7 -> 25.1, 26.2 -> 26.3).
  const bool alone = grid <= n_cu;
  float *esum = workspace;
  float *mref = workspace + (size_t)BH * M * 16 * MT;
  const float scale_log2 = 1.4426950408889634f / ((float)S * sqrtf((float)s.D));
#define HEART_AD_LAUNCH(DD, TT, BB)                                                                \
  do {                                                                                             \
    auto kern = antidiag_tile_kernel<DD, TT, BB>;                                                  \
    static DeviceFlags attr_set;                                                                   \
    if (hipError_t e = set_max_lds_once(attr_set, dev, reinterpret_cast<const void *>(kern),       \
                                        ad_lds(TT, BB)))                                           \
      return fail(HEART_EHIP, "hipFuncSetAttribute(antidiagonal tile kernel LDS): %s",             \
                  hipGetErrorString(e));                                                           \
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(2 * TT), ad_lds(TT, BB), st, (const uint16_t *)q, \
                       (const uint16_t *)k, s.q_stride[0], s.q_stride[1], s.q_stride[2],           \
                       s.k_stride[0], s.k_stride[1], s.k_stride[2], s.H, BH, s.N, S, M, MTQ, MT,   \
                       scale_log2, refresh, esum, mref);                                           \
  } while (0)
  if (s.D == 128) {
    if (few && alone)
      HEART_AD_LAUNCH(128, 128, 4);
    else if (few)
      HEART_AD_LAUNCH(128, 128, 2);
    else
      HEART_AD_LAUNCH(128, 256, 2);
  } else {
    if (few && alone)
      HEART_AD_LAUNCH(64, 128, 4);
    else if (few)
      HEART_AD_LAUNCH(64, 128, 2);
    else
      HEART_AD_LAUNCH(64, 256, 2);
  }
#undef HEART_AD_LAUNCH
  if (int rc = check_launch("antidiag_tile_kernel")) return rc;
  const dim3 cgrid((unsigned)((long long)BH * Nb));
  const size_t clds = (size_t)kAdKeysPerBlock * 16 * MT * sizeof(float);
  if (MT <= 16)
    hipLaunchKernelGGL(antidiag_combine_kernel<1>, cgrid, dim3(256), clds, st, Nb, M, MT, refresh, esum,
                       mref, scores);
  else if (MT <= 32)
    hipLaunchKernelGGL(antidiag_combine_kernel<2>, cgrid, dim3(256), clds, st, Nb, M, MT, refresh, esum,
                       mref, scores);
  else
    hipLaunchKernelGGL(antidiag_combine_kernel<4>, cgrid, dim3(256), clds, st, Nb, M, MT, refresh, esum,
                       mref, scores);
  return check_launch("antidiag_combine_kernel");
}

}  // namespace heart
