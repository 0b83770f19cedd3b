// heart_block_sparse_attn: softmax attention over the tokens of the kept key blocks of
// each query block (the sparse attention that consumes the top-p block mask; logits
// scaled by 1/sqrt(D) as in the appendix on query-key stability).
//
// Work decomposition: one workgroup per (b, h, query block); wavefront w of the
// workgroup owns query rows 32w .. 32w+31 of the block and loops over the kept
// key blocks with an online softmax.  Both contractions run on the bf16 matrix
// cores with v_mfma_f32_32x32x16_bf16, fp32 accumulation.
//
// The kernel computes TRANSPOSED tiles so that no accumulator ever has to move
// between lanes:
//   S^T (keys x queries) = K (keys x d) . Q^T (d x queries)
//   O^T (d x queries)   += V^T (d x keys) . P^T (keys x queries)
// In the 32x32 accumulator layout a lane holds one column (= one query, lane%32)
// and 16 rows (8*(r/4) + 4*(lane/32) + r%4, r = 0..15).  So every softmax
// statistic (running max, running sum, rescale factor) of a query lives in the two
// lanes l and l^32 and is a per-lane scalar, and the exponentiated S^T registers
// are, unchanged, the B operand of the second contraction: a lane must supply 8
// keys of its query per MFMA, and any assignment of keys to the 8 slots is valid
// as long as the A operand (V^T) uses the same one.
//
// K and V never pass through registers on their way in: they are copied from global
// memory straight into LDS by 16-byte LDS-direct buffer loads (rows past the end of the
// sequence are out of range for the buffer descriptor and arrive as zeros, with no
// branch and no address clamping).  Both tiles stay row-major [key][d] and unpadded (a
// direct load fills 1 KB of consecutive LDS); the 16-byte chunk index is XOR-swizzled
// with the row so that fragment reads are bank-conflict free.  K fragments are plain
// 16-byte reads; V^T fragments come from the transposing LDS read ds_read_b64_tr_b16.
//
// The kept key blocks are consumed as one stream of 32-key slices.  K and V arrive in
// double-buffered stages of 64 rows, loaded two slices ahead; V stages are skewed by one
// slice against K stages so that one workgroup barrier per 64 keys retires both (see the
// comment at the loop; D = 128 with blocks of 64 has stages of one slice, kStageRows).
// The softmax scale and log2(e) are folded into Q once (or applied to the logits, kExact), and
// the S^T accumulators start from minus the running reference exponent, so an
// accumulator goes into the exponential as it is.
//
// Scheduling.  Kept counts range from 1 to Nb per row and the densities of the heads
// differ a lot, the K/V of one head (16.8 MB at N = 32760, D = 128) is far larger than
// the 4 MB L2 of an XCD, and every query block re-reads its kept K/V blocks.  With a
// caller-provided workspace the launch therefore follows a plan (attn_plan.hip): whole
// heads are assigned to the 8 XCDs (greedily, heaviest head first, by total kept count),
// each XCD walks through its heads one at a time -- all its workgroups then share one
// head's K/V through that XCD's L2, and only 8 heads are in flight in the memory-side
// cache -- and inside a head the rows run in batches of similar kept lists (or, in a small
// workspace, the rows with the longest kept lists first).  A workgroup takes the next item
// of its XCD's list with an atomic counter; when that list is exhausted it takes from
// another XCD's list, which levels whatever imbalance the head assignment left.  Without a
// workspace an XCD works on a contiguous eighth of the query blocks of every head, in index
// order.  With fewer query blocks than places for workgroups the lists themselves are split
// (kSplit below).
#include <chrono>
#include <type_traits>

#include "heart_internal.h"

namespace heart {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(16))) float f32x16_t;
// Native vector types (not the HIP struct wrappers): loads and stores of these are
// first-class values, so staging arrays of them always live in registers.
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4_t;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;

union Frag8 {
  u32x4_t u;
  bf16x8_t v;
};

__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, b);
}

// buffer descriptor over one head's rows: offsets >= bytes read as zero
__device__ __forceinline__ __amdgpu_buffer_rsrc_t head_rsrc(const uint16_t *base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(base), 0, (int)bytes, 0x00020000);
}

// the same descriptor as four words in scalar registers, for hand-written buffer instructions
__device__ __forceinline__ u32x4_t head_rsrc_words(const uint16_t *base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  u32x4_t r;
  r.x = __builtin_amdgcn_readfirstlane((uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xffffu);
  r.z = __builtin_amdgcn_readfirstlane(bytes);
  r.w = 0x00020000u;
  return r;
}

// Key rows per K / V stage buffer: two 32-key slices, or one at D = 128, block 64.  There a workgroup
// has two wavefronts, and with stages of 64 rows (64 KB) the LDS of a CU holds two workgroups, one
// wavefront per SIMD; with 32 KB it holds four.  The price is a barrier per slice and loads that are one
// slice ahead instead of two; with two wavefronts per SIMD it is paid (N = 16384, 40 heads, 60 of 256
// blocks kept: 1764 -> 1289 us, 731 -> 1000 TFLOP/s; 4 blocks: 257 -> 193 us).
template <int D, int BLK>
constexpr int kStageRows = D == 128 && BLK == 64 ? 32 : 64;
// An XCD with no more heads than this walks their rows in turn: one after the other, the second
// head's long rows would start late and their length decide when the launch ends (12 heads at
// N = 32760: 1428 -> 1406 us for the whole step); with three heads the L2 sharing that this gives
// up costs more than it gains (24 heads at N = 119056: 33.1 -> 38.6 ms).
constexpr int kHeadsInTurn = 2;
// kExact (the default of the ABI): Q stays as it is and every logit is scaled in fp32 (one more
// multiply per logit); the error is then the bf16 rounding of the weights and of the output
// for any input scale.  !kExact (HEART_ATTN_FOLD_SCALE): the softmax scale is folded into Q
// once (one more bf16 rounding of the query; the error grows with the cube of the input scale,
// inside the budget for inputs of unit scale) and no per-logit multiply is left.
#ifndef HEART_ATTN_PF
#define HEART_ATTN_PF 4  // LDS fragment reads in flight ahead of the MFMAs
#endif
#ifndef HEART_ATTN_OCC
#define HEART_ATTN_OCC 2  // waves per SIMD the register budget is sized for
#endif

// Split rows.  A launch with fewer rows than the chip has places for workgroups (two per CU, four
// of the small ones at block 64) would leave the rest idle while each row walks its list
// alone; there S workgroups take a part of each list and write their unnormalised outputs, and
// attn_merge_kernel (or, of two parts, the second of them) adds them up.  S is as many as there are
// places for, with at least kSplitMinBlocks blocks a part where lists are full: a part costs about
// 10 us beside its blocks (launch, first loads, 64 KB written and read again), a block 0.8 us (64
// keys, D = 64) to 1.7 us (128 keys, D = 128).  All parts start at once, so such a launch needs no plan.  A function of the sizes only.
// Measured, whole call: dense 38 -> 19 us, a step at two heads of 16 rows 36 -> 31.5 us (which the
// host now bounds), steps of 100 to 250 rows 67 -> 33, 88 -> 38, 88 -> 43 us.
constexpr int kSplitCus = 256;        // CUs the places are counted for
constexpr int kSplitMinBlocks = 4;
constexpr int kSplitMax = 16;
constexpr int kLdsPerCu = 160 * 1024;
// floats of one wavefront's part: accumulators, reference exponent and row sum of every lane
template <int D>
constexpr int kPartFloats = 64 * (D / 2) + 128;
// Rows of few parts are added up by the workgroup that leaves the last of them (kSplitMerged, kSharedMerged).  That saves a
// launch, and of the two parts at a cut the one that ends later, mostly the end of a share, stays in registers: a 64 KB part
// (D = 128, block 128) is written and read once in the place of twice, which bound the launch (11.7 us for 512 cuts, 5.7
// TB/s).  It reads one part after the other, though, and the longest row of few has many: then a launch of a wavefront for 32
// columns of 32 rows is the faster way.  Steps and calls with the launch -> without, us: D = 128, block 128: 18 heads of 33
// rows (0.9 shares a row) 91.1 -> 85.1, two of 160 (1.6) 94.8 -> 91.9, two of 120 (2.1) 77.6 -> 77.3, one of 240 (2.1) 100 ->
// 101.7, one of 160 (3.2) 71 -> 76, two of five (3) 31.8 -> 29.7, six of six (4) 33.4 -> 34.5; D = 64, block 64: 20 of 101
// (0.5) 101 -> 96.4, one of 640 (1.6) 103.8 -> 103.3, one of 480 (2.1) 85.0 -> 88.6, four of 112 (2.3) 48.9 -> 54.1; two split
// parts, 18 of eleven 48.4 -> 44.9, 12 of 16 46.6 -> 41.9; four at D = 64, two of 16 21.9 -> 23.6.
constexpr int kMergeParts = 2;  // split rows
// (rows of fewer than eight blocks have four parts at most: seven blocks in parts of two)
constexpr bool merge_shares(long long n_share, long long rows, long long Nb) { return n_share < (Nb < 8 ? 4 : 2) * rows; }
constexpr float kNoKeys = -1.f;  // in the place of the row sum: a part without keys (a sum is not negative, but may be NaN)

// places for workgroups on the chip
static long long attn_places(int D, int block) {
  const int rows = D == 128 && block == 64 ? kStageRows<128, 64> : kStageRows<64, 64>;
  const int by_waves = HEART_ATTN_OCC * 4 / (block / 32), by_lds = kLdsPerCu / (4 * rows * D * 2);
  return (long long)kSplitCus * (by_waves < by_lds ? by_waves : by_lds);
}

int attn_split(long long BH, long long Nb, int D, int block) {
  const long long places = attn_places(D, block);
  if (BH > places || Nb > places) return 1;  // (beyond that their product can leave 64 bits)
  long long s = places / (BH * Nb);
  if (s > Nb / kSplitMinBlocks) s = Nb / kSplitMinBlocks;
  if (s > kSplitMax) s = kSplitMax;
  return s < 2 ? 1 : (int)s;
}

size_t attn_split_bytes(long long BH, long long Nb, int D, int block) {
  const int s = attn_split(BH, Nb, D, block);
  if (s == 1) return 0;
  const size_t part = D == 128 ? kPartFloats<128> : kPartFloats<64>;
  return (size_t)(BH * Nb) * s * (block / 32) * part * sizeof(float);
}

// Shared rows.  Where a place works on at most a few rows, their uneven lengths decide when a launch ends: the
// longest row alone takes as long as several of the mean.  Where the caller asks for it (workspace_bytes of
// heart_attn_balanced_workspace_bytes) lists are divided there, by one of three rules, and the rows that were
// are added up by the workgroup that leaves the last part, or by attn_merge_kernel (merge_shares):
//   shares  the kept blocks of all rows, row after row, are one sequence (lengths in half blocks) that is cut into equal
//           shares, one per place
//   parts   every row is split into parts of at most L blocks, L as small as the places allow; each workgroup has one
//           part, all start at once
//   whole   a workgroup per row, as far as that is no slower: few rows of nearly the same length
// Every workgroup finds the rule and its part or share from the kept counts by itself (read once, 16 KB at most): no plan and
// no queue, and what is divided where, and with it the bits, is a function of the counts alone.  Only the parts of a divided
// row are counted, by one ticket a row, where a workgroup adds them up.
// XCD x takes the x-th eighth of the parts or shares, so it sees an eighth of the heads.
// What it costs: 1.5 to 3 us until a workgroup knows its share, and the merge (2 to 4 us in the workgroups, 4 to 13 as a
// launch).  Calls with a plan -> with shares, lists of the timed fields, several seeds: 20 heads of 101 rows (D = 64, block 64)
// 99 to 127 -> 74 to 111 us; D = 128, block 128: six heads of 88 rows 193 to 224 -> 146 to 159, two of 247 375 -> 204 to 237;
// D = 128, block 64: 21 heads of 73 rows 110 to 118 -> 96; dense lists, four heads of 147 rows (D = 128, block 128) 726 -> 669.
constexpr int kShareGroup = 256, kShareMaxRows = 16 * kShareGroup;  // rows; counts are summed up in groups, four rows a lane
constexpr int kShareMin = 8;       // shortest share
constexpr int kSharePart = 2;      // fewest blocks of a part: a cut closer to an end of its row goes there
constexpr int kShareRowCost = 6;   // what a row costs beside its blocks (10 instead: 2 % slower over 30 shapes)
// The first workgroup of a CU is older than the others and its wavefronts go first: with equal shares it ends when the
// others have a fifth of theirs left (D = 64, block 64: 65 against 80 us), so its share is 1 + 1 / kShareOlder times as long.
constexpr int kShareOlder = 4;
// blocks of a row of `cnt` that lie before a cut `d` behind the start of the row
__device__ __forceinline__ int share_blocks(int d, int cnt) {
  const int e = min(max((d - kShareRowCost + 1) >> 1, 0), cnt);
  return e < kSharePart ? 0 : cnt - e < kSharePart ? cnt : e;
}

// Shares of a launch (workgroups; those that find no share for them end at once), 0 = rows are not shared.  A function
// of the sizes.  With a plan the uneven lengths cost the more the fewer rows a place has; with shares the workgroups of an
// XCD are at places of K/V that lie further apart than its L2 is wide, the more the longer the rows are.  Steps on lists of
// the timed fields (thresholds 0.85 to 0.98), plan -> shares, us:
//   up to 2.9 rows a place  D = 128, block 128: two heads of 520 rows (2.0) 815 -> 630, three of 360 (2.1) 767 -> 543, six
//                           of 230 (2.7) 588 -> 550, two of 700 (2.7) 1285 -> 1245, three of 480 (2.8) 1053 -> 909, five of
//                           300 (2.9) 843 -> 796; D = 64, block 64: 16 of 176 (2.8) 249 -> 181, six of 480 (2.8) 463 ->
//                           406; at 3 and 3.1: 11 of 140 398 -> 404, two of 800 1861 -> 1874
//   more, and rows a place times the elements of a head's keys up to share_near: D = 128: 16 of 110 (3.4) 406 -> 362, 21 of
//                           88 (3.6) 407 -> 362, 26 of 80 (4.1) 404 -> 371; beyond: 14 of 120 (3.3) 403 -> 419, 10 of 176
//                           (3.4) 511 -> 530, 12 of 256 (6) 1331 -> 1434; D = 64: 12 of 320 (3.8; block 64) 413 -> 377,
//                           eight of 248 (3.9; block 128) 666 -> 607, 14 of 160 (4.4) 467 -> 441; beyond: five of 400 (3.9)
//                           845 -> 845, 14 of 244 (6.7) 750 -> 790
//   D = 128, block 64       (four workgroups a CU feel the L2 most) two rows a place and share_near: two of 576 (1.1) 473 ->
//                           390, three of 480 (1.4) 450 -> 383, 14 of 128 (1.8) 173 -> 162; beyond: 30 of 122 (3.6) 286 -> 332
// Lists of 10 % of the blocks gain most (two of 700 rows 707 -> 522), for those that keep much see share_most.  Rows of few
// blocks a part of kSplitRows are left to that.
// (D = 64, block 64: heads of at most 64 blocks keep the limit of 2.5 rows a place, and with it the workspace size and the bits
// that the tests hold them to.  That is no limit of the chip: 52 heads of 49 rows, just below it, take 101 us with a plan and 74
// with shares, 41 of 64, just beyond, 110 and would take 82.)
// Dense lists need no levelling: only where a last round of whole rows would leave many places empty (D = 128, block 128:
// seven heads of 98 rows (1.3) 522 -> 508, six of 122 (1.4) 665 -> 673, two of 366 (1.4) 1936 -> 1987; D = 64: 12 of 147 (1.7)
// 382 -> 342, 20 of 147 (2.9) 591 -> 588).
// rows a place times elements of a head's keys
constexpr long long share_near(int D, int block) { return (D == 64 ? 650ll : block == 64 ? 700ll : 380ll) * 128 * 128; }

// Most kept blocks of a launch that are shared (kShareAny: any number).  Long lists in long rows gain nothing and lose: 0.88
// to 1 times as fast at D = 128, block 128, 0.84 at D = 64, block 64 with 950 rows a head, 0.7 to 0.95 at D = 128, block 64.
// Beyond share_sure the workgroups, which know all counts, therefore leave lists of more than 28 % of the blocks, or of more
// than share_far to a place, to a plan and a launch that follows it; where they do not, these two end at once (6 to 8 us).
// Calls of shares for any lists -> this, us, and with a plan: D = 128, block 128: two heads of 695 rows, 47 % kept, 3710 -> 3340
// (3327), 16 % 1166 -> 1179 (1190), three of 476, 70 % 3744 -> 3551 (3524), 14 % 713 -> 722 (906); D = 64, block 64: three of
// 951, 62 % 2940 -> 2305 (2298), 13 % 476 -> 483 (660); D = 128, block 64: three of 464, 68 % 1543 -> 1082 (1069), 13 % 259 ->
// 265 (338), eight of 226, 78 % 783 -> 712 (722), 15 % 156 -> 164 (229).
// Up to share_sure, and up to two rows a place (2.5 at D = 64, one at D = 128, block 64), any lists are shared: what lists that
// keep much lose there (up to 4 %; at most two rows a place up to a tenth, a fifth at D = 128, block 64) is little beside what
// others gain (1.1 to 1.6 times as fast), which the two launches would take a part of.  So with D = 64, block 128 for all (six
// heads of 293 rows 0.95 with 70 % kept, 1.06 with 37 %, 1.2 with 11 %).
// share_far: kept blocks a place.  An XCD that has rows of two heads at a time finds less of them in its L2.  Shares are
// as fast as the plan at, % of the blocks: D = 128, block 128: two heads of 695 rows 22, of 598 30, three of 476 15, of 415 28,
// of 354 29, four of 317 30, five of 256 27; D = 64, block 64: three of 951 15, of 854 17, four of 683 27, six of 464 31;
// D = 128, block 64: two of 537 29, three of 439 17, of 464 16, five of 287 31, six of 256 28.
constexpr long long share_sure(int D, int block) { return (D == 64 ? 430ll : block == 64 ? 150ll : 600ll) * 128 * 128; }
constexpr int share_far(int D, int block) { return D == 64 ? 380 : block == 64 ? 96 : 225; }
constexpr int kShareAny = 0x7fffffff;
static int share_most(long long BH, long long Nb, int D, int block) {
  const long long places = attn_places(D, block), rows = BH * Nb;
  if (D == 64 && block == 128) return kShareAny;
  if (2 * rows <= (D == 64 ? 5 : block == 64 ? 2 : 4) * places) return kShareAny;
  if (rows * Nb * D * block <= share_sure(D, block) * places) return kShareAny;
  const bool one_head = BH % kNumXcd == 0 || kNumXcd % BH == 0;  // an XCD has rows of one head at a time
  const long long all = rows * Nb * 7 / 25, far = (one_head ? 2 : 1) * share_far(D, block) * places;
  return (int)(all < far ? all : far);
}
int attn_shares(long long BH, long long Nb, int D, int block, bool dense) {
  const long long places = attn_places(D, block);
  if (BH > kShareMaxRows || Nb > kShareMaxRows || BH * Nb > kShareMaxRows) return 0;
  const long long rows = BH * Nb;
  const bool one = D == 128 && block == 64, near = rows * Nb * D * block <= share_near(D, block) * places;
  if (rows > places && one && (!near || rows > 2 * places)) return 0;
  if (10 * rows > 29 * places && !near) return 0;
  if (D == 64 && block == 64 && Nb <= 64 && 2 * rows > 5 * places) return 0;
  const int s = attn_split(BH, Nb, D, block);
  // Short rows in many parts each: what a workgroup takes to find its part costs more than even parts give.  Lists of the timed
  // fields, kSplitRows -> shares us: D = 64, block 64, one head of 167 rows (six parts) 19.8 -> 22.8, two of 115 (four) 23.7 -> 24.4,
  // but one of 197 (five) 28.5 -> 26.2, two of 165 (three) 31.4 -> 23.8; D = 128, block 64, three of 80 (four) 23.2 -> 26.1, two of
  // 105 (four) 27.6 -> 25.1, four of 77 (three) 37.3 -> 29.9; two parts, and blocks of 128, 1.0 to 2 times as fast from 15 on.
  const int few_blocks = block == 128 || s < 3 ? 15 : D == 64 ? 30 : s < 4 ? 15 : 24;  // a part
  if (s > 1 && (dense || Nb <= few_blocks * s)) return 0;
  if (dense && ((one && rows * Nb > 300 * places) || (rows > places && 8 * rows > (D == 64 ? 14 : 10) * places))) return 0;
  const long long most = rows * (Nb / kSharePart + 1);
  return (int)((most < places ? most : places) + kNumXcd - 1) / kNumXcd * kNumXcd;
}

// owners of divided rows (row, further parts, share) or tickets, then two parts per share: the one a share starts with and the
// one it ends with
size_t attn_share_bytes(long long BH, long long Nb, int D, int block, bool dense) {
  const int n = attn_shares(BH, Nb, D, block, dense);
  if (n == 0) return 0;
  const size_t part = D == 128 ? kPartFloats<128> : kPartFloats<64>;
  return (size_t)n * (sizeof(int4) + 2 * (size_t)(block / 32) * part * sizeof(float));
}

// Adds up the parts of rows where attn_kernel leaves that to a second launch: one wavefront per (32 query rows, 32 columns of
// the output), lanes as in attn_kernel.  Parts of item i are i * n_split .. ; of shared rows (`owner` given) the last part of share k
// and the first ones of the shares after it.  Bound by latency (the parts come from the L2s and the memory-side
// cache): four parts at a time.
template <int D, int BLK>
__global__ __launch_bounds__(D * 2) void attn_merge_kernel(const float *__restrict__ part, const int4 *__restrict__ owner,
                                                           int n_split, uint16_t *__restrict__ out, long long osb,
                                                           long long osh, long long osn, int H, int N, int Nb,
                                                           float *__restrict__ lse) {
  constexpr int NW = BLK / 32;
  const int lane = threadIdx.x & 63, dt = threadIdx.x >> 6, l32 = lane & 31, hf = lane >> 5;
  int item = (int)(blockIdx.x / NW);
  const int wave = (int)(blockIdx.x % NW);
  size_t first = (size_t)item * n_split, second = first + 1, step = 1;  // parts of the row
  if (owner) {
    const int4 own = owner[item];
    if (own.x < 0) return;
    first = 2 * (size_t)own.z + 1;
    second = first + 1;
    step = 2;
    item = own.x;
    n_split = own.y + 1;
  }
  auto part_of = [&](int s) -> const float * {
    s = min(s, n_split - 1);
    return part + ((s == 0 ? first : second + (size_t)(s - 1) * step) * NW + wave) * kPartFloats<D>;
  };
  const float ninf = -__builtin_inff();
  float m = ninf, l = 0.f;
  f32x4_t o[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) o[g] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < n_split; s0 += 4) {
    float ms[4], ls[4];
    f32x4_t x[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float *src = part_of(s0 + s);
      ms[s] = src[64 * (D / 2) + lane];
      ls[s] = src[64 * (D / 2) + 64 + lane];
      const f32x4_t *o4 = reinterpret_cast<const f32x4_t *>(src) + 4 * 64 * dt + lane;
#pragma unroll
      for (int g = 0; g < 4; ++g) x[s][g] = o4[64 * g];
      if (s0 + s >= n_split) ms[s] = ninf, ls[s] = kNoKeys;
    }
    const float m_old = m;
#pragma unroll
    for (int s = 0; s < 4; ++s) m = fmaxf(m, ms[s]);
    // (a part whose logits are all NaN or -inf keeps the reference -inf, like one without keys: its weight
    // is 0, but its sums count, because a NaN among them has to reach the result)
    const float m_fin = m == ninf ? 0.f : m;
    const float alpha = __builtin_amdgcn_exp2f(m_old - m_fin);
    l *= alpha;
#pragma unroll
    for (int g = 0; g < 4; ++g) o[g] *= alpha;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if (ls[s] == kNoKeys) continue;  // (accumulators of a part without keys are not written)
      const float w = __builtin_amdgcn_exp2f(ms[s] - m_fin);
      l = fmaf(ls[s], w, l);
#pragma unroll
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[g][e] = fmaf(x[s][g][e], w, o[g][e]);
    }
  }
  const int bh = item / Nb, qb = item % Nb, n = qb * BLK + wave * 32 + l32;
  const float l_tot = l + __shfl_xor(l, 32, 64);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (n >= N) return;
  if (lse && dt == 0 && hf == 0)
    lse[(size_t)bh * N + n] = l_tot > 0.f ? (m + log2f(l_tot)) * 0.6931471805599453f : ninf;
  uint16_t *dst = out + (bh / H) * osb + (bh % H) * osh + (long long)n * osn + 32 * dt + 4 * hf;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    u32x2_t pk;
    pk.x = cvt_pk_bf16(o[g][0] * inv, o[g][1] * inv);
    pk.y = cvt_pk_bf16(o[g][2] * inv, o[g][3] * inv);
    *reinterpret_cast<u32x2_t *>(dst + 8 * g) = pk;
  }
}

// Tickets of divided rows: `mark`, which no other call has, with the number of parts that are there in its lowest bits, so that
// memory of any contents is a ticket without parts.  The workgroup that finds all others there sets it back to zero: the
// next replay of a captured call has the same mark.
constexpr unsigned kMarkCount = 0xffff;
static_assert(kShareMaxRows <= (int)kMarkCount && kMergeParts == 2, "parts of a row");

// kMode: kPlanned, rows as a plan (or, without one, the workgroup's number) says; kSplitRows: a workgroup takes part of
// one row's list and leaves it in `part`; kSharedRows: a share of all rows
// kSplitMerged, kSharedMerged: the same, and the workgroup that leaves the last part of a row adds them up
// (instantiations of their own: with a branch at run time the others took 0.5 to 1 us longer; at D = 128 kSharedMerged keeps two
// registers in scratch memory while it adds up, behind the MFMA stream)
enum AttnMode { kPlanned, kSplitRows, kSharedRows, kSplitMerged, kSharedMerged };
template <int D, int BLK, bool kExact, AttnMode kMode>
__global__ __launch_bounds__(BLK * 2, HEART_ATTN_OCC) void attn_kernel(
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k,
    const uint16_t *__restrict__ v, uint16_t *__restrict__ out, long long qsb, long long qsh,
    long long qsn, long long ksb, long long ksh, long long ksn, long long vsb, long long vsh,
    long long vsn, long long osb, long long osh, long long osn, int H, int BH, int N, int Nb,
    const int *__restrict__ kept_idx, const int *__restrict__ kept_count, float scale_log2e,
    float *__restrict__ lse, int *__restrict__ plan, const int *__restrict__ seq, int *__restrict__ cursors,
    int cursor_step, float *__restrict__ part, int4 *__restrict__ owner,
    unsigned long long mark, int n_split, int n_few) {
  constexpr bool kSplit = kMode == kSplitRows || kMode == kSplitMerged, kShare = kMode == kSharedRows || kMode == kSharedMerged;
  constexpr bool kMerge = kMode == kSplitMerged || kMode == kSharedMerged;
  constexpr int NT = BLK * 2;            // threads
  constexpr int NW = NT / 64;            // wavefronts
  constexpr int DT = D / 32;             // 32-wide d tiles of the output
  constexpr int KS = D / 16;             // k-steps of the first contraction
  constexpr int CPR = D / 8;             // 16-byte chunks per token row
  constexpr int ROWB = D * 2;            // bytes of a token row in LDS (no padding)
  constexpr int RPB = 16 / CPR;          // rows per 256 bytes (one pass over the 64 banks)
  constexpr int SR = kStageRows<D, BLK>;
  constexpr bool kOne = SR == 32;        // stages of one slice
  constexpr int TILE_B = SR * ROWB;      // bytes of one K or V stage buffer
  constexpr int RPI = 64 / CPR;          // rows one LDS-direct load instruction covers
  constexpr int IPW = SR / RPI / NW;  // such instructions per wavefront and tile
  constexpr int NSL = BLK / 32;          // 32-key slices per key block
  constexpr int SO = D + 8;              // LDS row stride of the output staging (elements)
  // kExact: S^T comes out of the matrix cores in raw logit units and is multiplied by
  // scale * log2(e) in fp32 as soon as it is complete (in slots of the MFMA stream that have
  // VALU time to spare: where the maximum is folded), so that from there on both variants
  // hold logits in log2 units relative to the reference exponent.  The accumulators start
  // from -m_ref, which kExact therefore converts back to raw units (kInitScale).  The running
  // reference may lag the maximum by 8 log2 units.
  const float kInitScale = kExact ? 1.f / scale_log2e : 1.f;
  constexpr float kRescaleSlack = 8.f;
  static_assert(NW % 2 == 0 && IPW >= 1 && (NSL == 2 || NSL == 4), "tile layout");

  // LDS: [K stage 0][K stage 1][V stage 0][V stage 1], reused for the output at the end
  extern __shared__ __align__(1024) unsigned char smem[];
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)smem;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int l32 = lane & 31, hf = lane >> 5;

  // ---- state of the item (head, query block) being processed; set by begin_item ---------
  int bh = 0, qb = 0, b = 0, h = 0, qrow = 0, cnt = 0;
  const int *idx = kept_idx;
  __amdgpu_buffer_rsrc_t q_rs = head_rsrc(q, 0);
  u32x4_t k_rs = head_rsrc_words(k, 0), v_rs = head_rsrc_words(v, 0);
  const uint32_t k_row_bytes = (uint32_t)ksn * 2u, v_row_bytes = (uint32_t)vsn * 2u;

  // ---- per-lane constants of the LDS layout ---------------------------------------------
  // Chunk c (16 bytes) of tile row r is stored at chunk position c ^ f(r):
  //   K: f(r) = (r / RPB) % CPR      -- the 16 rows a quarter-wave reads with one
  //                                     ds_read_b128 (same chunk, consecutive rows) fall
  //                                     into 16 distinct 4-bank groups
  //   V: f(r) = 4 * ((r / RPB) % (CPR/4)) -- the 4 rows x 4 chunks that 32 lanes read with
  //                                     one transposing read fall into distinct groups
  // K fragment of k-step ks (A operand of S^T): row l32 of the slice, chunk 2 ks + hf.
  uint32_t koff[KS];
  {
    const int fk = (l32 / RPB) % CPR;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) koff[ks] = (uint32_t)(l32 * ROWB + (((2 * ks + hf) ^ fk) * 16));
  }
  // V^T fragment (A operand of O^T += V^T P^T) through ds_read_b64_tr_b16: within 16 lanes,
  // lane s supplies the address of 4 consecutive d of one key (key s/4, d chunk s%4) and
  // lane i receives d = i of keys 0..3.  A fragment (8 keys) is two such reads: keys
  // 16 s2 + 4 hf + 0..3 and 16 s2 + 8 + 4 hf + 0..3 of the slice, the order in which the
  // accumulator of S^T holds them.
  uint32_t voff[DT];
  {
    const int s = lane & 15, g16 = (lane >> 4) & 1;
    const int rowv = 4 * hf + (s >> 2);
    const int fv4 = (rowv / RPB) % (CPR / 4);
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      voff[dt] = (uint32_t)(rowv * ROWB + ((4 * (dt ^ fv4) + 2 * g16 + ((s & 3) >> 1)) * 16) +
                            (s & 1) * 8);
  }
  // LDS-direct loads: one instruction moves 16 bytes per lane to 1 KB of consecutive LDS
  // (RPI rows); lane l lands at chunk position l % CPR of row l / CPR and therefore fetches
  // global chunk (l % CPR) ^ f(row).  Wavefront w issues instructions w*IPW .. w*IPW+IPW-1
  // of a tile.  Rows past the end of the sequence are out of range for the descriptor and
  // arrive as zeros.
  uint32_t kdma[IPW], vdma;
  {
    const int drow = lane / CPR, dp = lane % CPR;
#pragma unroll
    for (int ii = 0; ii < IPW; ++ii) {
      const int r = (wave * IPW + ii) * RPI + drow;
      kdma[ii] = (uint32_t)drow * k_row_bytes + (uint32_t)((dp ^ ((r / RPB) % CPR)) * 16);
    }
    vdma = (uint32_t)drow * v_row_bytes + (uint32_t)((dp ^ (4 * ((drow / RPB) % (CPR / 4)))) * 16);
  }
  // tile `buf` of K (is_v = 0) or V (is_v = 1): instruction ii of this wavefront; the
  // first 32 rows of the tile come from key rows key_a.., the last 32 from key_b..
  auto dma = [&](int is_v, int ii, int buf, int key_a, int key_b) __attribute__((always_inline)) {
    const int half = kOne ? 0 : wave / (NW / 2), wi = kOne ? wave : wave % (NW / 2);
    const int krow = (half ? key_b : key_a) + (wi * IPW + ii) * RPI;
    const uint32_t voffset =
        is_v ? vdma + (uint32_t)krow * v_row_bytes : kdma[ii] + (uint32_t)krow * k_row_bytes;
    const uint32_t dst = smem_lds + (uint32_t)((2 * is_v + buf) * TILE_B + (wave * IPW + ii) * 1024);
    // (the compiler does not see this instruction's LDS write, so it adds no waits of
    // its own: completion is awaited explicitly before the barrier that publishes the tile.
    // The LDS destination travels in M0, which the statement saves and restores: the
    // compiler is free to keep values of its own there)
    uint32_t m0_saved;
    if (is_v)
      asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                   : "=&s"(m0_saved) : "s"(dst), "v"(voffset), "s"(v_rs) : "memory");
    else
      asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
                   "buffer_load_dwordx4 %2, %3, 0 offen lds\n\ts_mov_b32 m0, %0"
                   : "=&s"(m0_saved) : "s"(dst), "v"(voffset), "s"(k_rs) : "memory");
  };

  Frag8 qf[KS];      // Q fragments (B operand of S^T = K Q^T), kept in registers
  f32x16_t o[DT];    // O^T accumulators
  float m_ref = 0.f; // reference exponent (log2 domain) of the running sums
  // S^T accumulators start from -m_ref instead of zero, so they hold logits relative to
  // the reference exponent and go into the exponential as they are
  f32x16_t cinit;
  float l_run = 0.f;  // running sum over this lane's keys, relative to m_ref
  int split = 0;  // (split rows) which part of the kept list
  int e_begin = 0, e_end = 0, row_cnt = 0;  // (shared rows) part of the kept list, its length
  auto begin_item = [&](int item) __attribute__((always_inline)) {
    bh = item / Nb;
    qb = item % Nb;
    b = bh / H;
    h = bh % H;
    q_rs = head_rsrc(q + b * qsb + h * qsh, (uint32_t)(N * qsn * 2));
    k_rs = head_rsrc_words(k + b * ksb + h * ksh, (uint32_t)(N * ksn * 2));
    v_rs = head_rsrc_words(v + b * vsb + h * vsh, (uint32_t)(N * vsn * 2));
    qrow = qb * BLK + wave * 32 + l32;
    const uint32_t q_off = (uint32_t)qrow * ((uint32_t)qsn * 2u) + (uint32_t)hf * 16u;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      qf[ks].u = __builtin_amdgcn_raw_buffer_load_b128(q_rs, q_off + ks * 32, 0, 0);
    if constexpr (!kExact) {
      // fold the softmax scale and log2(e) into Q once: S^T then comes out of the matrix
      // cores in log2 units and no per-logit multiply is left on the VALU
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int w = 0; w < 4; ++w)
          qf[ks].u[w] = cvt_pk_bf16(bf16lo(qf[ks].u[w]) * scale_log2e, bf16hi(qf[ks].u[w]) * scale_log2e);
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
    m_ref = -__builtin_inff();
#pragma unroll
    for (int r = 0; r < 16; ++r) cinit[r] = 0.f;
    l_run = 0.f;
    const size_t row = (size_t)bh * Nb + qb;
    idx = kept_idx + row * Nb;
    if constexpr (kShare) {
      cnt = __builtin_amdgcn_readfirstlane(e_end - e_begin);
      idx += __builtin_amdgcn_readfirstlane(e_begin);
    } else {
      cnt = min(kept_count[row], Nb);
    }
    if constexpr (kSplit) {
      cnt = max(cnt, 0);
      const int per = (cnt + n_split - 1) / n_split, e0 = min(cnt, split * per);
      cnt = min(per, cnt - e0);
      idx += e0;
    }
  };

  // The kept blocks are consumed as one sequence of 32-key slices.  Kept indices are
  // clamped into [0, Nb) so that a bad list cannot leave the tensors; entries past the
  // end of the list repeat the last one (their data is never used).
  auto kept = [&](int e) -> int { return min(max(idx[min(max(e, 0), cnt - 1)], 0), Nb - 1); };
  // The loop body covers 4 slices starting at slice s0 (list entry eb) and looks ahead up
  // to slice s0+7: the block indices of entries eb .. eb+NE-1 are held in scalar registers
  // and advance by EPB entries per body.  New entries are loaded right before a barrier:
  // a scalar load can only be awaited together with all outstanding LDS reads, and there
  // the pipeline of LDS reads is drained anyway.
  constexpr int EPB = 4 / NSL;      // list entries per loop body
  constexpr int NE = 7 / NSL + 1;   // entries a body can refer to
  int jb[NE];
  // first key row of slice s0 + rel (rel = 0 .. 7) of the current body
  auto key_of = [&](int rel) -> int { return jb[rel / NSL] * BLK + (rel % NSL) * 32; };

  // ---- the stream of MFMAs -----------------------------------------------------------------
  // The kept key blocks are one sequence of 32-key slices sigma = 0, 1, ...  Per slice:
  //   B(sigma): S^T(sigma+1), KS MFMAs on K fragments; in their shadow the exponentials,
  //             bf16 rounding and row sum of slice sigma
  //   C(sigma): O^T += V^T P^T(sigma), NPV MFMAs on V^T fragments; in their shadow the
  //             maximum of S^T(sigma+1); the rare move of the reference exponent follows
  // K and V arrive in stages of 64 rows (two slices), double-buffered, by LDS-direct
  // loads that are issued two slices before their first use.  K stage i holds slices
  // (2i, 2i+1), V stage i holds slices (2i-1, 2i): with this skew the last read of a K
  // stage (in B(2i)) and of a V stage (in C(2i)) are adjacent, ONE barrier per two slices
  // retires both, and every B phase has an S^T to overlap its exponentials with.
  //   ... B(2i) C(2i) | wait for own loads, barrier | B(2i+1) [issue stage i+2] C(2i+1) ...
  // The loop body covers 4 slices (2 stages) so that buffer indices are constants.  Every
  // MFMA takes its A operand from a ring of PF registers filled by LDS reads that run PF
  // stream positions ahead, across phases and the loop back-edge; only the barriers
  // restart the ring.  The instruction order written here is the intended issue order.
  constexpr int NPV = 2 * DT;             // MFMAs of one slice's O^T update
  constexpr int STEP = KS + NPV;
  constexpr int SEQ = 4 * STEP;
  constexpr int G_B0 = STEP, G_B1 = 3 * STEP;  // stream positions right after the barriers
  // (stages of one slice: K and V stage i hold slice i, and a barrier follows every slice)
  constexpr int PF = HEART_ATTN_PF < KS ? HEART_ATTN_PF : KS;
  static_assert(!kOne || NSL == 2, "stages of one slice: blocks of two");
  static_assert(16 % KS == 0 && SEQ % PF == 0 && PF <= KS && PF <= NPV, "stream layout");

  // A-operand fragment of stream position g.  Slice q (0..3) of the body: its V and the
  // K of slice q+1 both live in buffer ((q+1)/2)%2, rows ((q+1)%2)*32.
  auto fetch = [&](int g) __attribute__((always_inline)) -> u32x4_t {
    g %= SEQ;
    const int n = g / STEP + 1, r = g % STEP;
    const int buf = kOne ? (r < KS ? n : n - 1) & 1 : (n >> 1) & 1, row0 = kOne ? 0 : (n & 1) * 32;
    if (r < KS)
      return *reinterpret_cast<const u32x4_t *>(smem + buf * TILE_B + row0 * ROWB + koff[r]);
    const int m = r - KS;
    const unsigned char *p = smem + (2 + buf) * TILE_B + (row0 + 16 * (m / DT)) * ROWB + voff[m % DT];
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4_t *)(p));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) s16x4_t *)(p + 8 * ROWB));
    const u32x2_t a = __builtin_bit_cast(u32x2_t, lo), c = __builtin_bit_cast(u32x2_t, hi);
    return u32x4_t{a.x, a.y, c.x, c.y};
  };
  Frag8 ring[PF];
  auto prefetch_after = [&](int g) __attribute__((always_inline)) {
    const int t2 = g + PF;
    const bool crosses = kOne ? t2 / STEP != g / STEP : (g < G_B0 && t2 >= G_B0) || (g < G_B1 && t2 >= G_B1);
    if (!crosses) ring[t2 % PF].u = fetch(t2);
  };
  auto refill = [&](int g0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < PF; ++j) ring[(g0 + j) % PF].u = fetch(g0 + j);
  };

  f32x16_t sacc[2];  // S^T of the slice being exponentiated and of the next one
  Frag8 pf[2];       // P^T of the current slice: [s2] = rows 8*s2 .. 8*s2+7 of the accumulator

  // Weights of one slice: exp2 of the accumulator (already relative to the reference
  // exponent), rounded to bf16 for the second contraction; the row sum adds the unrounded
  // fp32 weights.  The 8 element pairs of a lane are 24 micro-ops (exponential,
  // exponential, convert + row sum) that are pinned, a few at a time, behind MFMAs: only
  // about 24 cycles of a wave's own VALU work hide behind one of its MFMAs, and a slot
  // that exceeds that stalls the matrix pipeline.
  float xt0 = 0.f, xt1 = 0.f;  // the pair in flight
  auto exp_uop = [&](const f32x16_t &x, int u) __attribute__((always_inline)) {
    const int r = 2 * (u / 3), st = u % 3;
    // (the empty asm statements pin each result to its slot: without them the compiler
    // sinks the whole computation to its first use, out of the MFMA shadow)
    if (st == 0) {
      xt0 = __builtin_amdgcn_exp2f(x[r]);
      asm volatile("" : "+v"(xt0));
    } else if (st == 1) {
      xt1 = __builtin_amdgcn_exp2f(x[r + 1]);
      asm volatile("" : "+v"(xt1));
    } else {
      // (plain adds for the row sum: they co-issue with MFMAs, dot instructions do not)
      uint32_t pk = cvt_pk_bf16(xt0, xt1);
      l_run += xt0 + xt1;
      asm volatile("" : "+v"(pk), "+v"(l_run));
      pf[r / 8].u[(r % 8) / 2] = pk;
    }
  };
  constexpr int UB = 16 / KS;        // micro-ops per B slot (16 of the 24 in B)
  constexpr int UC = 8 / DT;         // micro-ops per C slot m < DT (the other 8)
  // B: S^T into sacc[dst], stream positions g0 .. g0+KS-1, with the weights of the slice in
  // sacc[dst ^ 1] interleaved.  extra(slot) injects the loads of a later stage.
  auto qk_step = [&](int dst, int g0, auto &&extra) __attribute__((always_inline)) {
    f32x16_t acc;
    const f32x16_t &prev = sacc[dst ^ 1];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[(g0 + ks) % PF].v, qf[ks].v,
                                                    ks == 0 ? cinit : acc, 0, 0, 0);
      prefetch_after(g0 + ks);
#pragma unroll
      for (int u = 0; u < UB; ++u) exp_uop(prev, ks * UB + u);
      extra(ks);
      __builtin_amdgcn_sched_barrier(0);
    }
    sacc[dst] = acc;
  };
  // keys at or past row `nvalid` of the slice (end of a ragged last key block) get no weight
  auto mask_slice = [&](f32x16_t &x, int nvalid) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = 8 * (r >> 2) + 4 * hf + (r & 3);
      if (key >= nvalid) x[r] = -__builtin_inff();
    }
  };
  // maximum of one accumulator over this lane's 16 keys, in 4 partial steps so that it
  // can be spread over MFMA slots; step i folds elements 4i .. 4i+3
  auto max_part = [&](const f32x16_t &x, int i, float m) __attribute__((always_inline)) -> float {
    m = fmaxf(fmaxf(m, x[4 * i]), x[4 * i + 1]);       // v_max3_f32
    return fmaxf(fmaxf(m, x[4 * i + 2]), x[4 * i + 3]);  // v_max3_f32
  };
  // After the maximum m_rel of a slice (over this lane's keys, relative to the reference
  // exponent): the reference only moves when some logit exceeds it by more than the slack,
  // so exponentials stay below 2^slack and almost every slice takes the short path (one
  // compare per lane and a wave-wide vote).  The long path combines the two lanes of each
  // query (lane l and l^32, one v_permlane32_swap), moves the reference of the queries
  // that need it, rescales their sums, makes the not yet exponentiated slice x relative to
  // the new reference, and rewrites the accumulator start values.  A slice whose keys are
  // all past the end has maximum -inf and never moves the reference.
  auto finish_max = [&](float m_rel, f32x16_t &x) __attribute__((always_inline)) {
    const bool first = m_ref == -__builtin_inff();
    if (__any(m_rel > kRescaleSlack || (first && m_rel > -__builtin_inff()))) {
      uint32_t sw0, sw1;
      swap_halves32(__float_as_uint(m_rel), sw0, sw1);
      m_rel = fmaxf(__uint_as_float(sw0), __uint_as_float(sw1));
      const bool bump = m_rel > kRescaleSlack || (first && m_rel > -__builtin_inff());
      const float base = first ? 0.f : m_ref;       // what the accumulators are relative to
      const float delta = bump ? m_rel : 0.f;
      const float m_new = bump ? base + m_rel : m_ref;
      const float alpha = bump ? __builtin_amdgcn_exp2f(m_ref - m_new) : 1.f;  // 0 the first time
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
#pragma unroll
      for (int r = 0; r < 16; ++r) x[r] -= delta;
      m_ref = m_new;
      const float c0 = m_ref == -__builtin_inff() ? 0.f : -m_ref * kInitScale;
#pragma unroll
      for (int r = 0; r < 16; ++r) cinit[r] = c0;
    }
  };
  // C: O^T += V^T P^T of the slice in sacc[cur], stream positions g0 .. g0+NPV-1.  The first DT slots
  // finish the weights of the slice (consumed by the second half of the MFMAs); the second half of the
  // slots folds the maximum of sacc[cur ^ 1], whose MFMAs were issued before this phase and have drained
  // by then.
  auto pv_step = [&](int cur, int g0) __attribute__((always_inline)) -> float {
    float m_loc = -__builtin_inff();
    f32x16_t &nx = sacc[cur ^ 1];
    const f32x16_t &cx = sacc[cur];
#pragma unroll
    for (int m = 0; m < NPV; ++m) {
      o[m % DT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[(g0 + m) % PF].v, pf[m / DT].v, o[m % DT], 0, 0, 0);
      prefetch_after(g0 + m);
      if (m < DT) {
#pragma unroll
        for (int u = 0; u < UC; ++u) exp_uop(cx, 16 + m * UC + u);
      }
      if (m >= DT) {
#pragma unroll
        for (int i = 0; i < 4 / DT; ++i) {
          const int part = (m - DT) * (4 / DT) + i;
          if constexpr (kExact) {
#pragma unroll
            for (int e = 0; e < 4; ++e) nx[4 * part + e] *= scale_log2e;  // raw logits -> log2 units
          }
          m_loc = max_part(nx, part, m_loc);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    return m_loc;
  };
  auto no_extra = [](int) {};
  auto wait_loads_and_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  };

  // ---- work loop --------------------------------------------------------------------------
  // With a plan the workgroups are persistent (two per CU): each takes items from the list
  // of its XCD (workgroup ids are dealt round-robin to the XCDs; one head: all from list 0) and,
  // once that list is empty, from the other XCDs' lists.  The first item of a workgroup is the
  // one its number among the workgroups of its list names; the plan starts the cursors behind those, so the
  // launch does not begin with hundreds of atomics on one cache line.  Without a plan a
  // workgroup processes the one item its id maps to.
  __shared__ int s_item;
  const int x0 = (int)(blockIdx.x % kNumXcd);
  int n_wg = (int)gridDim.x;  // workgroups that take items
  if constexpr (kOne && kMode == kPlanned)
    if (plan && n_few < n_wg) {
      long long kept = 0;
      for (int i = 0; i < BH; ++i) kept += plan[kPlanHdr + BH + i];
      n_wg = working_groups(n_wg, n_few, kept, BH, Nb);
      if ((int)blockIdx.x >= n_wg) return;
    }
  const int own = BH == 1 ? 0 : x0;  // own list
  const int len0 = plan ? plan[kNumXcd + own] : 0;
  const int off0 = plan ? plan[2 * kNumXcd + own] : 0;
  // entry i of a list of `len` items whose heads start at off_x in the head table: the heads one
  // after the other, or, where a list has few of them, their rows in turn
  const int *head_tbl = plan + kPlanHdr;
  auto entry = [&](int off_x, int len, int i) -> int {
    const int nh = len / Nb;
    const bool in_turn = nh <= kHeadsInTurn;
    const int r = in_turn ? i % nh : i / Nb, p = in_turn ? i / nh : i - r * Nb;
    return seq[head_tbl[off_x + r] * Nb + p];
  };
  const int n_own = list_first(n_wg, own, BH);  // workgroups of this list
  int i_own = (int)(BH == 1 ? blockIdx.x : blockIdx.x / kNumXcd);  // (wavefront 0) last entry taken from the own list
  // (wavefront 0) an item of the own list, else of the list whose next item is the longest, else
  // -1.  Lanes 0..7 look at the eight cursors at once and an atomic goes only to a list that still
  // has items: same-address atomics of all XCDs are served one after another (about 40 ns each),
  // and a workgroup that asked every empty list before it ended made the end of each launch a
  // queue of 8 atomics per workgroup -- 300 us at 1024 workgroups (D = 64, block 64, N = 6417,
  // 20 heads: 406 -> 90 us), 150 us at 512.
  auto take = [&]() -> int {
    const int x = (own + lane) % kNumXcd;
    const int len = lane < kNumXcd ? plan[kNumXcd + x] : 0;
    const int off = lane < kNumXcd ? plan[2 * kNumXcd + x] : 0;
    unsigned long long asked = 0;
    for (;;) {
      uint32_t key = 0;  // kept blocks of the list's next item (own list: first), lane; 0 = empty
      if (lane < kNumXcd && !((asked >> lane) & 1)) {
        const int cur = __hip_atomic_load(&cursors[x * cursor_step], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur < len) {
          const int n = lane == 0 ? Nb : min(max(kept_count[entry(off, len, cur)], 0), Nb);
          key = (uint32_t)(n + 1) * kNumXcd + (uint32_t)(kNumXcd - 1 - lane);
        }
      }
      HEART_WAVE_REDUCE(uint32_t, key, HEART_OP_UMAX);
      if (key == 0) return -1;
      const int l = kNumXcd - 1 - (int)(key % kNumXcd);
      asked |= 1ull << l;  // (a list that turns out to be empty is not asked again)
      const int xs = (own + l) % kNumXcd;
      int i = 0;
      if (lane == 0) i = atomicAdd(&cursors[xs * cursor_step], 1);
      i = __builtin_amdgcn_readfirstlane(i);
      if (i < plan[kNumXcd + xs]) {
        if (l == 0) i_own = i;
        return entry(plan[2 * kNumXcd + xs], plan[kNumXcd + xs], i);
      }
    }
  };
  int item = -1;
  // (shared rows) which share (or part), start of the row in the sequence, end of the share, parts of the row (0 = shares)
  int share = 0, row0 = 0, cut1 = 0, parts = 0;
  // boundary k of n shares: evenly, or, where every place has one, by XCD and with older shares 1 + 1 / kOlder times as
  // long as the others (in steps of 1 / 256; the last of an XCD takes what the division leaves)
  constexpr int kPlacesXcd = kSplitCus / kNumXcd * 8 / NW, kOldXcd = kSplitCus / kNumXcd, kOlder = kShareOlder;
  int cut_step = 0, cut_rest = 0;
  bool tiers = false;
  auto share_cut = [&](int k) __attribute__((always_inline)) -> int {
    if (!tiers) return k * cut_step + min(k, cut_rest);
    const int x = k / kPlacesXcd, s = k % kPlacesXcd;  // (cut_rest: length of the sequence)
    return x * (cut_rest / kNumXcd) + min(x, cut_rest % kNumXcd) + ((s * cut_step + min(s, kOldXcd) * (cut_step / kOlder)) >> 8);
  };
  auto next_row = [&]() __attribute__((always_inline)) {
    row0 += 2 * row_cnt + kShareRowCost;
    ++item;
    e_begin = 0;
    row_cnt = min(max(kept_count[min(item, BH * Nb - 1)], 0), Nb);
  };
  // the part of the row that belongs to this share; false if the share ends before it (a cut at the start of a
  // row leaves it to the next share, also one without blocks)
  auto in_share = [&]() __attribute__((always_inline)) -> bool {
    if (parts) return true;
    const int end = row0 + 2 * row_cnt + kShareRowCost;
    e_end = cut1 < end ? share_blocks(cut1 - row0, row_cnt) : row_cnt;
    return cut1 > row0 && (cut1 >= end || e_end > e_begin);
  };
  if constexpr (kShare) {
    constexpr int kGroups = kShareMaxRows / kShareGroup, GPW = kGroups / NW;
    // groups a wavefront has of as many rows as places
    constexpr int PG = (kNumXcd * kPlacesXcd + kShareGroup * NW - 1) / (kShareGroup * NW);
    __shared__ int group_sum[2][kGroups];
    __shared__ int wave_longest[NW];
    __shared__ int found[4];
    const int rows = BH * Nb;
    // counts of four rows a lane, group i * NW + wave, zero past the end (out of range for the descriptor).  No
    // branches: a branch to code that is not in the instruction cache yet costs as much as the work it saves.
    int c[GPW][4];
    {
      const __amdgpu_buffer_rsrc_t rs = head_rsrc(reinterpret_cast<const uint16_t *>(kept_count), (uint32_t)rows * 4u);
#pragma unroll
      for (int i = 0; i < GPW; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          c[i][j] = (int)__builtin_amdgcn_raw_buffer_load_b32(rs, ((i * NW + wave) * kShareGroup + 4 * lane + j) * 4, 0, 0);
      int sum[GPW];
#pragma unroll
      for (int i = 0; i < GPW; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j) c[i][j] = min(max(c[i][j], 0), Nb);
        sum[i] = c[i][0] + c[i][1] + c[i][2] + c[i][3];
      }
#pragma unroll
      for (int i = 0; i < GPW; ++i) sum[i] = wave_sum_i32(sum[i]);
      // (the longest row is asked for where there are no more rows than places: the first PG groups)
      int longest = 0;
#pragma unroll
      for (int i = 0; i < PG; ++i) longest = max(longest, max(max(c[i][0], c[i][1]), max(c[i][2], c[i][3])));
      longest = (int)wave_max_u32((uint32_t)longest);
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < GPW; ++i) group_sum[0][i * NW + wave] = sum[i];
        wave_longest[wave] = longest;
      }
    }
    __syncthreads();
    int gl = lane < kGroups ? group_sum[0][lane] : 0;  // blocks of group `lane`, then its length
    const int blocks = __builtin_amdgcn_readfirstlane(wave_sum_i32(gl)), total = 2 * blocks + kShareRowCost * rows, n_wg = (int)gridDim.x;
    if constexpr (kMode == kSharedMerged) {
      // (n_few: the most blocks that are shared; *cursors: whether the plan is to do it)
      if (cursors && blockIdx.x == 0 && t == 0)
        __hip_atomic_store(cursors, blocks > n_few ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (blocks > n_few) return;
    }
    // blocks of a part, 0 = shares.  Any number from blocks / (n_wg - rows) up gives no more parts than workgroups
    // (n / most + 1 a row).  The rule is the one with the shortest way, in half blocks: the longest row; a part and
    // the merge of all; a share with a row more than the mean and the merge (which takes one for 64 parts).
    int most = 0;
    if (rows <= n_wg) {
      int longest = 0;
#pragma unroll
      for (int i = 0; i < NW; ++i) longest = max(longest, wave_longest[i]);
      const float per_wg = __builtin_amdgcn_rcpf((float)n_wg);
      const int t_shares = (int)((float)total * per_wg) + kShareRowCost + 2 + n_wg / 64;
      int t_parts = 0x7fffffff;
      if (rows < n_wg) {
        most = max((int)((float)blocks * __builtin_amdgcn_rcpf((float)(n_wg - rows)) * 1.00001f) + 1, kSharePart);
        t_parts = 2 * most + 2 + (int)(((float)blocks * __builtin_amdgcn_rcpf((float)most) + (float)rows) * (1.f / 64.f));
      }
      // (rows that walk through long lists together find each other's K/V in the L2; four workgroups a CU feel it most)
      const int t_whole = 2 * longest - longest / (kOne ? 4 : 8);
      if (t_shares < t_parts) most = 0;
      if (t_whole <= min(t_shares, t_parts)) most = max(longest, 1);
      most = __builtin_amdgcn_readfirstlane(most);
    }
    // length of a row of n blocks in the sequence: its parts, or half blocks
    const float len_a = most ? __builtin_amdgcn_rcpf((float)most) : 2.f;
    const float len_b = most ? (float)(most - 1) * len_a : (float)kShareRowCost;
    const int len_cap = most ? 1 : 0x7fffffff;
    auto row_len = [&](int n, bool is_row) __attribute__((always_inline)) -> int {
      const int len = min(max((int)fmaf((float)n, len_a, len_b), 1), max(n, len_cap));
      return is_row ? len : 0;
    };
    if (most) {
#pragma unroll
      for (int i = 0; i < PG; ++i) {
        int sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) sum += row_len(c[i][j], (i * NW + wave) * kShareGroup + 4 * lane + j < rows);
        sum = wave_sum_i32(sum);
        if (lane == 0) group_sum[1][i * NW + wave] = sum;
      }
      __syncthreads();
      gl = lane < PG * NW ? group_sum[1][lane] : 0;
    } else {
      gl = 2 * gl + kShareRowCost * min(max(rows - lane * kShareGroup, 0), kShareGroup);
    }
    const int gs = wave_scan_i32(gl);
    const int n_share = most ? __builtin_amdgcn_readlane(gs, 63) : min(n_wg, max(total / kShareMin, 1));
    tiers = !most && n_share == kNumXcd * kPlacesXcd;
    if (tiers) {
      cut_step = (int)((uint32_t)(total / kNumXcd * 256) / (uint32_t)(kPlacesXcd + kOldXcd / kOlder));
      cut_rest = total;
    } else {
      cut_step = most ? 1 : (int)((uint32_t)total / (uint32_t)n_share);
      cut_rest = most ? 0 : total - cut_step * n_share;
    }
    const int s0 = x0 * n_share / kNumXcd, s1 = (x0 + 1) * n_share / kNumXcd;
    share = s0 + (int)(blockIdx.x / kNumXcd);
    const int cut0 = share_cut(share);
    cut1 = share_cut(share + 1);
    // the row that the share starts in: found by the wavefront that holds its group
    const int g = __popcll(__ballot(gs <= cut0));
    const int g0 = g ? __builtin_amdgcn_readlane(gs, g - 1) : 0;
    if (share < s1 && g % NW == wave) {
      const int r0 = g * kShareGroup + 4 * lane;
      int l[4], n[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        n[j] = c[0][j];
#pragma unroll
        for (int i = 1; i < GPW; ++i)
          if (i == g / NW) n[j] = c[i][j];
        l[j] = row_len(n[j], r0 + j < rows);
      }
      const int sum = l[0] + l[1] + l[2] + l[3];
      int end = g0 + wave_scan_i32(sum), at = end - sum;  // rows of this lane: at .. end
      if (at <= cut0 && cut0 < end) {
        int j = 0, len = l[0], cnt_j = n[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) {
          const bool later = j == i - 1 && cut0 >= at + len;
          at = later ? at + len : at;
          len = later ? l[i] : len;
          cnt_j = later ? n[i] : cnt_j;
          j = later ? i : j;
        }
        found[0] = r0 + j;
        found[1] = at;
        found[2] = cnt_j;
        found[3] = len;
      }
    }
    __syncthreads();
    item = __builtin_amdgcn_readfirstlane(found[0]);
    row0 = __builtin_amdgcn_readfirstlane(found[1]);
    row_cnt = __builtin_amdgcn_readfirstlane(found[2]);
    if (most) {
      parts = __builtin_amdgcn_readfirstlane(found[3]);
      e_begin = (share - row0) * row_cnt / parts;
      e_end = (share - row0 + 1) * row_cnt / parts;
    } else {
      e_begin = share_blocks(cut0 - row0, row_cnt);
    }
    if (!kMerge && t == 0) owner[blockIdx.x] = int4{-1, 0, 0, 0};
    if (share >= s1) return;
    if (!parts && e_begin > 0 && e_begin == row_cnt) next_row();
  } else if (kMode == kPlanned && plan) {
    if (i_own < len0) {
      item = __builtin_amdgcn_readfirstlane(entry(off0, len0, i_own));
    } else {
      if (wave == 0) {
        const int it = take();
        if (lane == 0) s_item = it;
      }
      __syncthreads();
      item = __builtin_amdgcn_readfirstlane(s_item);
    }
  } else if constexpr (kSplit) {
    // XCD x takes the x-th eighth of the parts: by head, part of the list and query block, so that
    // its workgroups share the K/V of one part of one head
    const int n = BH * Nb * n_split, per = (n + kNumXcd - 1) / kNumXcd, slot = (int)(blockIdx.x / kNumXcd);
    const int w = x0 * per + slot;
    if (slot < per && w < n) {
      split = w / Nb % n_split;
      item = w / (Nb * n_split) * Nb + w % Nb;
    }
  } else {
    // XCD x takes the x-th eighth of the query blocks of every head, heads in order
    const int per = (Nb + kNumXcd - 1) / kNumXcd;  // query blocks per XCD and head
    const long long slot = blockIdx.x / kNumXcd;
    const int qb0 = x0 * per + (int)(slot % per);
    if (qb0 < Nb) item = (int)(slot / per) * Nb + qb0;  // else: padding of the last eighth
  }
  // (kMerge) The parts of a row are n, this one is number `mine`; the first is that of share k0.  The end of a share is mostly the
  // last part of its row: if the others are there this one stays in registers.  (Asked while the last loads are awaited.)
  int n = n_split, mine = split, k0 = share;
  bool last = false;
  auto ticket = [&]() __attribute__((always_inline)) -> unsigned long long * {
    // (one reference exponent per query: the upper half of its 64 places in a row's first part holds the row's ticket)
    return kShare ? reinterpret_cast<unsigned long long *>(owner + k0)
                  : reinterpret_cast<unsigned long long *>(part + (size_t)item * n_split * NW * kPartFloats<D> + 64 * 16 * DT + 32);
  };
  auto arrived = [&](unsigned long long v) __attribute__((always_inline)) -> int {
    return (v & ~(unsigned long long)kMarkCount) == mark && (int)(v & kMarkCount) < n ? (int)(v & kMarkCount) : 0;
  };
  // (an empty part, cnt = 0, comes from split rows only)
  auto partial = [&]() __attribute__((always_inline)) -> bool { return kSplit || (kShare && e_end - e_begin < row_cnt); };
  auto find_parts = [&]() __attribute__((always_inline)) {
    last = false;
    if constexpr (kShare) {
      if (parts) {
        n = parts;
        mine = share - row0;
        k0 = row0;
      } else {
        k0 = share;
        while (share_blocks(share_cut(k0) - row0, row_cnt) > 0) --k0;
        mine = share - k0;
        n = mine + 1;
        // (a part has two blocks at least, so the row has two: cuts behind it give all of its blocks, and the loop ends)
        for (int k = share + 1; share_blocks(share_cut(k) - row0, row_cnt) < row_cnt; ++k) ++n;
      }
      n = __builtin_amdgcn_readfirstlane(n);
      k0 = __builtin_amdgcn_readfirstlane(k0);
      mine = __builtin_amdgcn_readfirstlane(mine);
      if (mine == 0) {
        if (t == 0) s_item = arrived(__hip_atomic_load(ticket(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == n - 1;
        last = true;  // (if s_item says so)
      }
    }
  };
  while (kShare ? in_share() : item >= 0 && item < BH * Nb) {
  if constexpr (kMode == kSharedMerged) item = __builtin_amdgcn_readfirstlane(item);
  begin_item(item);
  // (thread 0) cursor value and item id of the NEXT item.  The cursor is advanced only in
  // the last loop body, not earlier: items are then started in list order up to about a
  // microsecond, and neighbouring rows of a head, whose kept lists overlap, walk through
  // K/V together (reserving the next item a whole row ahead costs a third of the L2 hits).
  int i_next = -1, item_next = -1;
  // (only while every workgroup of the list can expect another item of the own list: the last
  // round looks at the cursors first, so that it ends without a queue of failing atomics)
  const bool ahead = kMode == kPlanned && plan && i_own + n_own < len0;

  if (cnt > 0) {
    // ---- prologue: stages 0 and 1 in flight, S^T and maximum of slice 0 --------------------
    {
#pragma unroll
      for (int e = 0; e < NE; ++e) jb[e] = kept(e);
      const int k0 = key_of(0), k1 = key_of(1), k2 = key_of(2), k3 = key_of(3);
#pragma unroll
      for (int ii = 0; ii < IPW; ++ii) dma(0, ii, 0, k0, k1);
#pragma unroll
      for (int ii = 0; ii < IPW; ++ii) dma(1, ii, 0, k0, k0);
      if constexpr (kOne) {
#pragma unroll
        for (int ii = 0; ii < IPW; ++ii) dma(0, ii, 1, k1, k1);
        wait_loads_and_barrier();
      } else {
#pragma unroll
        for (int ii = 0; ii < IPW; ++ii) dma(0, ii, 1, k2, k3);
#pragma unroll
        for (int ii = 0; ii < IPW; ++ii) dma(1, ii, 1, k1, k2);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * IPW) : "memory");  // stage 0 has landed
        __syncthreads();
      }
      f32x16_t acc = cinit;  // zeros: no reference exponent yet
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        Frag8 a;
        a.u = fetch(3 * STEP + ks);  // K of slice 0: buffer 0, rows 0
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, qf[ks].v, acc, 0, 0, 0);
      }
      if constexpr (kExact) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] *= scale_log2e;
      }
      sacc[0] = acc;
      const int nv = N - k0;
      if (nv < 32) mask_slice(sacc[0], nv);
    }
    float m_loc = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < 4; ++i) m_loc = max_part(sacc[0], i, m_loc);
    finish_max(m_loc, sacc[0]);
    if constexpr (kOne) __syncthreads();  // K of slice 0 has been read
    refill(0);

    const int T = cnt * NSL / 2;  // pairs of slices
    if constexpr (kOne) {
      // stages of one slice: while slice s is worked on, K of slice s+2 goes to the buffer that
      // slice s left and V of slice s+1 to that of slice s-1
      auto one_slice = [&](auto j_const) __attribute__((always_inline)) {
        constexpr int j = decltype(j_const)::value;  // slice s0 + j of the body
        const int kn = key_of(j + 2), vn = key_of(j + 1);
        qk_step((j + 1) & 1, j * STEP, [&](int ks) {
#pragma unroll
          for (int ii = 0; ii < 2 * IPW; ++ii)
            if (ii * KS / (2 * IPW) == ks) {
              if (ii < IPW) dma(0, ii, j & 1, kn, kn);
              else dma(1, ii - IPW, (j + 1) & 1, vn, vn);
            }
        });
        const int nv = N - vn;
        if (nv < 32) mask_slice(sacc[(j + 1) & 1], nv);
        m_loc = pv_step(j & 1, j * STEP + KS);
        finish_max(m_loc, sacc[(j + 1) & 1]);
      };
      for (int st = 0; st < T; st += 2) {
        int jn[EPB];
        one_slice(std::integral_constant<int, 0>{});
#pragma unroll
        for (int i = 0; i < EPB; ++i) jn[i] = kept(2 * st / NSL + NE + i);
        wait_loads_and_barrier();
#pragma unroll
        for (int i = 0; i < EPB; ++i) asm volatile("" : "+s"(jn[i]));  // loaded before the barrier
        if (ahead && t == 0 && st + 2 >= T) i_next = atomicAdd(&cursors[own * cursor_step], 1);
        refill(STEP);
        one_slice(std::integral_constant<int, 1>{});
        if (st + 1 >= T) break;
        wait_loads_and_barrier();
        refill(2 * STEP);
        one_slice(std::integral_constant<int, 2>{});
        wait_loads_and_barrier();
        refill(3 * STEP);
        one_slice(std::integral_constant<int, 3>{});
        wait_loads_and_barrier();
        refill(0);
        // advance the entry window
#pragma unroll
        for (int e = 0; e + EPB < NE; ++e) jb[e] = jb[e + EPB];
#pragma unroll
        for (int i = 0; i < EPB; ++i) jb[NE - EPB + i] = jn[i];
      }
    } else
    for (int st = 0; st < T; st += 2) {
      // (body: slices s0 = 2 st .. s0+3, list entry eb = s0 / NSL)
      int jn[EPB];
      // ---- slice s0: B, C, then the barrier that retires K stage st and V stage st ----
      qk_step(1, 0, no_extra);
      {
        const int nv = N - key_of(1);
        if (nv < 32) mask_slice(sacc[1], nv);
      }
      m_loc = pv_step(0, KS);
      finish_max(m_loc, sacc[1]);
#pragma unroll
      for (int i = 0; i < EPB; ++i) jn[i] = kept(2 * st / NSL + NE + i);
      wait_loads_and_barrier();
#pragma unroll
      for (int i = 0; i < EPB; ++i) asm volatile("" : "+s"(jn[i]));  // loaded before the barrier
      if (ahead && t == 0 && st + 2 >= T) i_next = atomicAdd(&cursors[own * cursor_step], 1);
      refill(G_B0);
      // ---- slice s0+1; stage st+2 -> buffers 0 ----
      {
        const int ka = key_of(4), kb = key_of(5), va = key_of(3);
        qk_step(0, STEP, [&](int ks) {
#pragma unroll
          for (int ii = 0; ii < 2 * IPW; ++ii)
            if (ii * KS / (2 * IPW) == ks) {
              if (ii < IPW) dma(0, ii, 0, ka, kb);
              else dma(1, ii - IPW, 0, va, ka);
            }
        });
      }
      {
        const int nv = N - key_of(2);
        if (nv < 32) mask_slice(sacc[0], nv);
      }
      m_loc = pv_step(1, STEP + KS);
      finish_max(m_loc, sacc[0]);
      if (NSL == 2 && st + 1 >= T) break;
      // ---- slice s0+2: B, C, barrier retiring K stage st+1 and V stage st+1 ----
      qk_step(1, 2 * STEP, no_extra);
      {
        const int nv = N - key_of(3);
        if (nv < 32) mask_slice(sacc[1], nv);
      }
      m_loc = pv_step(0, 2 * STEP + KS);
      finish_max(m_loc, sacc[1]);
      wait_loads_and_barrier();
      refill(G_B1);
      // ---- slice s0+3; stage st+3 -> buffers 1 ----
      {
        const int ka = key_of(6), kb = key_of(7), va = key_of(5);
        qk_step(0, 3 * STEP, [&](int ks) {
#pragma unroll
          for (int ii = 0; ii < 2 * IPW; ++ii)
            if (ii * KS / (2 * IPW) == ks) {
              if (ii < IPW) dma(0, ii, 1, ka, kb);
              else dma(1, ii - IPW, 1, va, ka);
            }
        });
      }
      {
        const int nv = N - key_of(4);
        if (nv < 32) mask_slice(sacc[0], nv);
      }
      m_loc = pv_step(1, 3 * STEP + KS);
      finish_max(m_loc, sacc[0]);
      // advance the entry window
#pragma unroll
      for (int e = 0; e + EPB < NE; ++e) jb[e] = jb[e + EPB];
#pragma unroll
      for (int i = 0; i < EPB; ++i) jb[NE - EPB + i] = jn[i];
    }
    if constexpr (kMerge)
      if (partial()) find_parts();
    // loads of stages past the end may still be in flight towards LDS
    wait_loads_and_barrier();
  }
  if (ahead && wave == 0) {
    if (lane == 0 && i_next < 0) i_next = atomicAdd(&cursors[own * cursor_step], 1);  // (row without kept blocks)
    i_next = __builtin_amdgcn_readfirstlane(i_next);
    if (i_next < len0) {
      i_own = i_next;
      item_next = entry(off0, len0, i_next);
    }
  }

  if (!kMerge && partial()) {
    // ---- part of a row: unnormalised output and its softmax state, as the lanes hold them ----
    const int slot = kShare ? 2 * share + (e_begin == 0) : item * n_split + split;
    float *dst = part + ((size_t)slot * NW + wave) * kPartFloats<D>;
    dst[64 * 16 * DT + lane] = m_ref;
    dst[64 * 16 * DT + 64 + lane] = cnt > 0 ? l_run : kNoKeys;
    if (cnt > 0) {
      f32x4_t *o4 = reinterpret_cast<f32x4_t *>(dst);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g)
          o4[(4 * dt + g) * 64 + lane] = f32x4_t{o[dt][4 * g], o[dt][4 * g + 1], o[dt][4 * g + 2], o[dt][4 * g + 3]};
    }
    if (kShare && e_begin == 0 && t == 0) {
      int more = max(parts - 1, 1);
      for (int k = share + 2; !parts; ++k) {
        const int d = share_cut(k) - row0;
        if (d >= 2 * row_cnt + kShareRowCost || share_blocks(d, row_cnt) == row_cnt) break;
        ++more;
      }
      owner[blockIdx.x] = int4{item, more, share, 0};
    }
    if (kSplit || parts || e_end < row_cnt) break;
    next_row();
    continue;
  }

  if constexpr (kMerge) if (partial()) {
    // ---- the same part, or, if the others are there, their sum -------------------------------
    constexpr int kAgent = 16;  // (sc1: past the L2 of this XCD, where the workgroups of all XCDs meet)
    constexpr int kStateB = 64 * 16 * DT * 4;  // byte offset of the state behind the accumulators
    auto part_rsrc = [&](int s) __attribute__((always_inline)) -> __amdgpu_buffer_rsrc_t {
      const int slot = kShare ? 2 * (k0 + s) + (s == 0) : item * n_split + s;
      return head_rsrc(reinterpret_cast<const uint16_t *>(part + (size_t)slot * NW * kPartFloats<D>),
                       (uint32_t)(NW * kPartFloats<D> * sizeof(float)));
    };
    uint32_t ln = (uint32_t)lane;
    asm volatile("" : "+v"(ln));  // (offsets made here: kept through the MFMA stream they would cost it registers)
    const uint32_t part_off = (uint32_t)(wave * kPartFloats<D> * sizeof(float)) + 16u * ln;
    const uint32_t state_off = (uint32_t)(wave * kPartFloats<D> * sizeof(float)) + (uint32_t)kStateB + 4u * ln;
    const uint32_t ref_off = state_off - 4u * (ln & 32u);
    last = last && __builtin_amdgcn_readfirstlane(s_item) != 0;
    if (!last) {
      const __amdgpu_buffer_rsrc_t dst = part_rsrc(mine);
      if (ln < 32u) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(m_ref), dst, ref_off, 0, kAgent);
      __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(cnt > 0 ? l_run : kNoKeys), dst, state_off + 256u, 0, kAgent);
      if (cnt > 0) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int g = 0; g < 4; ++g) {
            const f32x4_t x = {o[dt][4 * g], o[dt][4 * g + 1], o[dt][4 * g + 2], o[dt][4 * g + 3]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, x), dst,
                                                   part_off + (uint32_t)((4 * dt + g) * 1024), 0, kAgent);
          }
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (t == 0) {
        unsigned long long v = __hip_atomic_load(ticket(), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int c;
        do {
          c = arrived(v);
        } while (!__hip_atomic_compare_exchange_strong(ticket(), &v, mark | (unsigned long long)(c + 1), __ATOMIC_RELAXED,
                                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        s_item = c == n - 1;
      }
      __syncthreads();
      last = __builtin_amdgcn_readfirstlane(s_item) != 0;
      __syncthreads();
    }
    if (!last) {
      if (kSplit || parts || e_end < row_cnt) break;
      next_row();
      continue;
    }
    if (t == 0) __hip_atomic_store(ticket(), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // ---- the last part of a row: the sum of all, in their order whichever was the last --------
    // One of two parts, or the first, stays in the registers; else this one too is read again (one more array of accumulators does
    // not fit the registers).  (A part whose logits are all NaN or -inf keeps the reference -inf: its weight is 0, but its sums
    // count, because a NaN among them has to reach the result.)
    f32x16_t x[DT];
    float ms, ls;
    auto load_part = [&](int s) __attribute__((always_inline)) {
      const __amdgpu_buffer_rsrc_t src = part_rsrc(s);
      ms = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src, ref_off, 0, kAgent));
      ls = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(src, state_off + 256u, 0, kAgent));
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4_t y = __builtin_bit_cast(
              f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(src, part_off + (uint32_t)((4 * dt + g) * 1024), 0, kAgent));
#pragma unroll
          for (int e = 0; e < 4; ++e) x[dt][4 * g + e] = y[e];
        }
    };
    // (accumulators of a part without keys are not written)
    auto has_keys = [&](float sum) -> bool {
      return __builtin_amdgcn_readfirstlane(__float_as_int(sum)) != __float_as_int(kNoKeys);
    };
    if (kSplit || n == 2) {
      load_part(1 - mine);
      if (has_keys(ls)) {
        // (products rounded on their own: their sum does not depend on which of the two is the own part)
#pragma clang fp contract(off)
        const float m_new = fmaxf(m_ref, ms), m_fin = m_new == -__builtin_inff() ? 0.f : m_new;
        const float w = __builtin_amdgcn_exp2f(m_ref - m_fin), wx = __builtin_amdgcn_exp2f(ms - m_fin);
        l_run = l_run * w + ls * wx;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] = o[dt][r] * w + x[dt][r] * wx;
        m_ref = m_new;
      }
    } else {
      if (mine != 0) {
        m_ref = -__builtin_inff();
        l_run = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
      }
      for (int s = mine == 0 ? 1 : 0; s < n; ++s) {
        load_part(s);
        if (!has_keys(ls)) continue;
        const float m_new = fmaxf(m_ref, ms), m_fin = m_new == -__builtin_inff() ? 0.f : m_new;
        const float alpha = __builtin_amdgcn_exp2f(m_ref - m_fin), w = __builtin_amdgcn_exp2f(ms - m_fin);
        l_run = fmaf(ls, w, l_run * alpha);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] = fmaf(x[dt][r], w, o[dt][r] * alpha);
        m_ref = m_new;
      }
    }
  }

  // ---- epilogue: normalise, stage through LDS, coalesced bf16 store -----------------------
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (lse && hf == 0 && qrow < N)
    lse[(size_t)bh * N + qrow] =
        l_tot > 0.f ? (m_ref + log2f(l_tot)) * 0.6931471805599453f : -__builtin_inff();
  uint16_t *sO = reinterpret_cast<uint16_t *>(smem);  // [BLK][SO]
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      u32x2_t pk;
      pk.x = cvt_pk_bf16(o[dt][4 * g + 0] * inv, o[dt][4 * g + 1] * inv);
      pk.y = cvt_pk_bf16(o[dt][4 * g + 2] * inv, o[dt][4 * g + 3] * inv);
      *reinterpret_cast<u32x2_t *>(sO + (wave * 32 + l32) * SO + dt * 32 + 8 * g + 4 * hf) = pk;
    }
  __syncthreads();
  uint16_t *obase = out + b * osb + h * osh;
  constexpr int OCH = (BLK * CPR) / NT;  // 16-byte chunks of the output per thread
  constexpr int O_R_STEP = NT / CPR;
  const int o_r0 = t / CPR, o_c = (t % CPR) * 8;
#pragma unroll
  for (int it = 0; it < OCH; ++it) {
    const int r = o_r0 + it * O_R_STEP;
    const int n = qb * BLK + r;
    if (n < N)
      *reinterpret_cast<u32x4_t *>(obase + (long long)n * osn + o_c) =
          *reinterpret_cast<const u32x4_t *>(sO + r * SO + o_c);
  }
  if constexpr (kShare) {
    if (parts) break;
    next_row();
    __syncthreads();  // everyone has read the output staging before the next row's loads
    continue;
  }
  if (kSplit || !plan) break;
  if (wave == 0) {
    if (item_next < 0) item_next = take();
    if (lane == 0) s_item = item_next;
  }
  __syncthreads();  // also: everyone has read the output staging before the next item's loads
  item = __builtin_amdgcn_readfirstlane(s_item);
  }  // work loop
}

// A mark that no other call has (kMarkCount: its low bits are zero): counted from a place that the clock and the address space
// of the process choose.
static unsigned long long call_mark() {
  static std::atomic<unsigned long long> next{0};
  unsigned long long m = next.load(std::memory_order_relaxed);
  if (m == 0) {
    unsigned long long x = (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() ^
                           (unsigned long long)reinterpret_cast<uintptr_t>(&next);
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;  // (the finaliser of SplitMix64, Steele et al. 2014)
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    next.compare_exchange_strong(m, ((x ^ (x >> 31)) & ~(unsigned long long)kMarkCount) | (kMarkCount + 1ull));
  }
  return next.fetch_add(kMarkCount + 1ull, std::memory_order_relaxed);
}

template <int D, int BLK, bool kExact>
static int launch_attn_t(const heart_shape &s, const void *q, const void *k, const void *v,
                         const int *kept_idx, const int *kept_count, float scale, void *out,
                         float *lse, int *order, size_t order_bytes, hipStream_t st) {
  const int Nb = (s.N + BLK - 1) / BLK;
  const int BH = s.B * s.H;
  const long long n_items = (long long)BH * Nb;
  const int n_split = order ? attn_split(BH, Nb, D, BLK) : 1;
  const int n_share = order ? attn_shares(BH, Nb, D, BLK, false) : 0;
  // (exactly that size asks for shares: a larger buffer kept for several shapes is one that knows nothing of them)
  const bool share = n_share > 0 && order_bytes == attn_balanced_bytes(BH, Nb, D, BLK, false);
  const bool split = !share && n_split > 1 && order_bytes >= attn_split_bytes(BH, Nb, D, BLK);
  const size_t lds = 4 * (size_t)kStageRows<D, BLK> * D * 2;  // >= BLK * (D + 8) * 2 of the output staging
  const bool merged = (share && merge_shares(n_share, n_items, Nb)) || (split && n_split <= kMergeParts);
  const int most = share && merged ? share_most(BH, Nb, D, BLK) : kShareAny;
  const bool watch = most != kShareAny;  // (more rows than places: always merged)
  const int dev = current_device();
  if (dev < 0) return fail(HEART_EHIP, "heart_block_sparse_attn: cannot identify the current device");
  const float sc = scale > 0.f ? scale : 1.0f / sqrtf((float)D);
  const float scale_log2e = sc * 1.4426950408889634f;
  float *part = nullptr;
  int4 *owner = nullptr;
  auto run = [&](auto mode, long long grid, int *plan, const int *seq, int *cursors, int cursor_step, int n_few) -> int {
    auto kern = attn_kernel<D, BLK, kExact, decltype(mode)::value>;
    static DeviceFlags attr_set;  // per instantiation: the attribute is per function and device
    if (hipError_t e = set_max_lds_once(attr_set, dev, reinterpret_cast<const void *>(kern), (int)lds))
      return fail(HEART_EHIP, "hipFuncSetAttribute(max dynamic LDS %zu): %s", lds, hipGetErrorString(e));
    if (grid > 0x7fffffffLL) return fail(HEART_EUNSUPPORTED, "heart_block_sparse_attn: grid too large");
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(BLK * 2), lds, st,
                       (const uint16_t *)q, (const uint16_t *)k, (const uint16_t *)v,
                       (uint16_t *)out, s.q_stride[0], s.q_stride[1], s.q_stride[2], s.k_stride[0],
                       s.k_stride[1], s.k_stride[2], s.v_stride[0], s.v_stride[1], s.v_stride[2],
                       s.o_stride[0], s.o_stride[1], s.o_stride[2], s.H, BH, s.N, Nb, kept_idx,
                       kept_count, scale_log2e, lse, plan, seq, cursors, cursor_step, part, owner,
                       merged ? call_mark() : 0ull, n_split, n_few);
    return check_launch("attn_kernel");
  };
  auto merge = [&](long long n) -> int {
    hipLaunchKernelGGL((attn_merge_kernel<D, BLK>), dim3((unsigned)(n * (BLK / 32))), dim3(D * 2), 0, st, part,
                       owner, n_split, (uint16_t *)out, s.o_stride[0], s.o_stride[1], s.o_stride[2], s.H, s.N, Nb, lse);
    return check_launch("attn_merge_kernel");
  };
  const int *skip = nullptr;  // (a plan for lists that the shares left)
  if (share) {
    owner = reinterpret_cast<int4 *>(order);
    part = reinterpret_cast<float *>(owner + n_share);
    int *left = watch ? order + 2 : nullptr;  // (the third word of the first owner is free beside its ticket)
    if (int rc = merged ? run(std::integral_constant<AttnMode, kSharedMerged>{}, n_share, nullptr, nullptr, left, 1, most)
                        : run(std::integral_constant<AttnMode, kSharedRows>{}, n_share, nullptr, nullptr, nullptr, 1, 0))
      return rc;
    if (!watch) return merged ? HEART_OK : merge(n_share);
    skip = left;
    order = reinterpret_cast<int *>(part);  // (the parts are not there where there is a plan)
    order_bytes -= (size_t)n_share * sizeof(int4);
  }
  if (split) {
    part = reinterpret_cast<float *>(order);
    const long long grid = (n_items * n_split + kNumXcd - 1) / kNumXcd * kNumXcd;
    if (merged) return run(std::integral_constant<AttnMode, kSplitMerged>{}, grid, nullptr, nullptr, nullptr, 1, 0);
    if (int rc = run(std::integral_constant<AttnMode, kSplitRows>{}, grid, nullptr, nullptr, nullptr, 1, 0)) return rc;
    return merge(n_items);
  }
  const std::integral_constant<AttnMode, kPlanned> planned;
  if (!order)
    return run(planned, (long long)BH * ((Nb + kNumXcd - 1) / kNumXcd) * kNumXcd, nullptr, nullptr, nullptr, 1, 0);
  // persistent workgroups: as many as are resident at once (HEART_ATTN_OCC per SIMD, i.e.
  // two workgroups of four wavefronts per CU)
  const int n_cu = cu_count(dev);
  if (n_cu <= 0) return fail(HEART_EHIP, "heart_block_sparse_attn: cannot query the number of CUs");
  const long long resident = (long long)n_cu * HEART_ATTN_OCC * 4 / (BLK / 32);
  const long long grid = n_items < resident ? n_items : resident;
  const bool few = kStageRows<D, BLK> < 64 && BH <= kFewHeads && n_items <= kFewRows && grid > 2 * n_cu;
  const int n_few = few ? 2 * n_cu : (int)grid;  // (see working_groups)
  const int *seq = nullptr;
  int *spread = nullptr;
  if (int rc = launch_attn_plan(BH, Nb, (int)grid, n_few, (int)n_items, kept_idx, kept_count, skip, order, order_bytes,
                                &seq, &spread, st))
    return rc;
  return run(planned, grid, order, seq, spread ? spread : order, spread ? kCursorSpread : 1, n_few);
}

template <bool kExact>
static int launch_attn_e(const heart_shape &s, const void *q, const void *k, const void *v,
                         const int *kept_idx, const int *kept_count, float scale, void *out,
                         float *lse, int *order, size_t order_bytes, hipStream_t st) {
  if (s.D == 128 && s.block == 128)
    return launch_attn_t<128, 128, kExact>(s, q, k, v, kept_idx, kept_count, scale, out, lse, order, order_bytes, st);
  if (s.D == 128 && s.block == 64)
    return launch_attn_t<128, 64, kExact>(s, q, k, v, kept_idx, kept_count, scale, out, lse, order, order_bytes, st);
  if (s.D == 64 && s.block == 128)
    return launch_attn_t<64, 128, kExact>(s, q, k, v, kept_idx, kept_count, scale, out, lse, order, order_bytes, st);
  if (s.D == 64 && s.block == 64)
    return launch_attn_t<64, 64, kExact>(s, q, k, v, kept_idx, kept_count, scale, out, lse, order, order_bytes, st);
  return fail(HEART_EUNSUPPORTED, "heart_block_sparse_attn: unsupported (D, block) = (%d, %d)",
              s.D, s.block);
}

int launch_attn(const heart_shape &s, const void *q, const void *k, const void *v,
                const int *kept_idx, const int *kept_count, float scale, unsigned flags, void *out,
                float *lse, int *order, size_t order_bytes, hipStream_t st) {
  // the kernel addresses one head's rows through 32-bit buffer offsets
  const long long lim = 0xffffffffLL;
  const long long rows = (long long)s.N + 2 * s.block;  // staging may address a few rows past N
  if (rows * s.q_stride[2] * 2 > lim || rows * s.k_stride[2] * 2 > lim ||
      rows * s.v_stride[2] * 2 > lim)
    return fail(HEART_EUNSUPPORTED,
                "heart_block_sparse_attn: (N + 2*block) * token stride * 2 bytes must stay "
                "below 4 GiB");
  if (flags & HEART_ATTN_FOLD_SCALE)
    return launch_attn_e<false>(s, q, k, v, kept_idx, kept_count, scale, out, lse, order, order_bytes, st);
  return launch_attn_e<true>(s, q, k, v, kept_idx, kept_count, scale, out, lse, order, order_bytes, st);
}

// ---- launch plan in static device memory, for callers that cannot allocate --------------------
// One array per GPU (every device the library runs on holds its own copy at its own address
// until the process ends).  In host code the array's name is only a stand-in for the symbol:
// the device address is looked up once per device, with that device current, and only that
// pointer is handed to kernels.
static __device__ __align__(256) int g_plan_scratch[HEART_ATTN_STATIC_PLAN_BYTES / sizeof(int)];

int attn_static_plan(int **ptr) {
  const int dev = current_device();
  if (dev < 0)
    return fail(HEART_EHIP, "heart_block_sparse_attn_static: cannot identify the current device");
  static std::atomic<int *> addr[kMaxDevices];
  int *p = addr[dev].load(std::memory_order_acquire);
  if (!p) {
    void *sym = nullptr;
    const hipError_t e = hipGetSymbolAddress(&sym, HIP_SYMBOL(g_plan_scratch));
    if (e != hipSuccess || !sym)
      return fail(HEART_EHIP, "heart_block_sparse_attn_static: hipGetSymbolAddress: %s",
                  hipGetErrorString(e));
    p = static_cast<int *>(sym);
    addr[dev].store(p, std::memory_order_release);  // (threads that race store the same address)
  }
  *ptr = p;
  return HEART_OK;
}

}  // namespace heart
