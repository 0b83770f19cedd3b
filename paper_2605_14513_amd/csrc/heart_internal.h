// Internal helpers shared by the HIP translation units of libheart (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "heart.h"
#include "heart_diag.h"

namespace heart {

// Records a message for heart_last_error() and returns `code`.
int fail(int code, const char *fmt, ...);
void clear_error();
// Checks hipGetLastError() after a launch; returns HEART_OK or HEART_EHIP.
int check_launch(const char *what);

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool stride_ok(const long long s[3]) {
  // strides are in 2-byte elements; 16-byte granularity = multiples of 8 elements
  return s[0] % 8 == 0 && s[1] % 8 == 0 && s[2] % 8 == 0 && s[2] > 0;
}

// bf16 pair packed in a 32-bit word -> two fp32
__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// fp32 -> bf16 bits, round to nearest even (inputs are finite here)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

// Lane exchanges on the VALU.  v_permlane16_swap / v_permlane32_swap exchange the odd
// rows (upper half) of their first operand with the even rows (lower half) of the
// second.  Fed the same value twice they return the pair (r0, r1) with
//   swap16: r0 = rows (0,0,2,2), r1 = rows (1,1,3,3) of v     (a row is 16 lanes)
//   swap32: r0 = halves (lo, lo), r1 = halves (hi, hi) of v
// so OP(r0, r1) combines every lane with its partner row / half, identically on both
// sides.  The second operand goes through an empty asm so that the compiler cannot
// see that both operands are the same value (it would then fold r0 and r1 into one).
__device__ __forceinline__ void swap_rows16(uint32_t v, uint32_t &r0, uint32_t &r1) {
  uint32_t w = v;
  asm volatile("" : "+v"(w));
  const auto r = __builtin_amdgcn_permlane16_swap(v, w, false, false);
  r0 = r[0];
  r1 = r[1];
}
__device__ __forceinline__ void swap_halves32(uint32_t v, uint32_t &r0, uint32_t &r1) {
  uint32_t w = v;
  asm volatile("" : "+v"(w));
  const auto r = __builtin_amdgcn_permlane32_swap(v, w, false, false);
  r0 = r[0];
  r1 = r[1];
}

// Wave-wide reductions that leave the result in every lane, on the VALU only (no LDS
// round trips): xor-1 and xor-2 inside quads and rotations by 4 and 8 inside rows of 16
// lanes as DPP modifiers, then the row and half exchanges above.
#define HEART_WAVE_REDUCE(T, v, OP)                                                      \
  do {                                                                                   \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0xB1, 0xf, 0xf, false))); /* quad_perm [1,0,3,2] */ \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0x4E, 0xf, 0xf, false))); /* quad_perm [2,3,0,1] */ \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0x124, 0xf, 0xf, false))); /* row_ror:4 */ \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0x128, 0xf, 0xf, false))); /* row_ror:8 */ \
    {                                                                                    \
      uint32_t r0_, r1_;                                                                 \
      swap_rows16(__builtin_bit_cast(uint32_t, v), r0_, r1_);                            \
      v = OP(__builtin_bit_cast(T, r0_), __builtin_bit_cast(T, r1_));                    \
    }                                                                                    \
    {                                                                                    \
      uint32_t r0_, r1_;                                                                 \
      swap_halves32(__builtin_bit_cast(uint32_t, v), r0_, r1_);                          \
      v = OP(__builtin_bit_cast(T, r0_), __builtin_bit_cast(T, r1_));                    \
    }                                                                                    \
  } while (0)
// The same reduction over each half (32 lanes) of the wavefront separately: the result of
// lanes 0..31 in every lane of 0..31, that of lanes 32..63 in every lane of 32..63.
#define HEART_HALF_REDUCE(T, v, OP)                                                      \
  do {                                                                                   \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0xB1, 0xf, 0xf, false)));          \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0x4E, 0xf, 0xf, false)));          \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0x124, 0xf, 0xf, false)));         \
    v = OP(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(                          \
                  0u, __builtin_bit_cast(uint32_t, v), 0x128, 0xf, 0xf, false)));         \
    {                                                                                    \
      uint32_t r0_, r1_;                                                                 \
      swap_rows16(__builtin_bit_cast(uint32_t, v), r0_, r1_);                            \
      v = OP(__builtin_bit_cast(T, r0_), __builtin_bit_cast(T, r1_));                    \
    }                                                                                    \
  } while (0)
// (functions, not expression macros: each argument -- a DPP read -- must be evaluated
// exactly once and with all lanes active)
__device__ __forceinline__ uint32_t heart_op_umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ __forceinline__ uint32_t heart_op_umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
#define HEART_OP_ADD(a, b) ((a) + (b))
#define HEART_OP_FMAX(a, b) fmaxf((a), (b))
#define HEART_OP_UMAX(a, b) heart_op_umax((a), (b))
#define HEART_OP_UMIN(a, b) heart_op_umin((a), (b))

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  HEART_WAVE_REDUCE(uint32_t, v, HEART_OP_ADD);
  return v;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  HEART_WAVE_REDUCE(uint32_t, v, HEART_OP_UMAX);
  return v;
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t v) {
  HEART_WAVE_REDUCE(uint32_t, v, HEART_OP_UMIN);
  return v;
}
// Inclusive prefix sum over the wavefront: shifts by 1, 2, 4, 8 inside rows of 16 lanes, then the last lane
// of rows 0 and 2, then of the lower half, added to the lanes behind it.
__device__ __forceinline__ int wave_scan_i32(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31
  return v;
}
__device__ __forceinline__ int wave_sum_i32(int v) { return (int)wave_sum_u32((uint32_t)v); }
__device__ __forceinline__ uint32_t half_sum(uint32_t v) {
  HEART_HALF_REDUCE(uint32_t, v, HEART_OP_ADD);
  return v;
}
// Sum of per-lane masses below 2^40: two 32-bit reductions over the low 20 bits and the
// rest (each stays below 2^32), recombined exactly.
__device__ __forceinline__ unsigned long long half_sum(unsigned long long v) {
  uint32_t lo = (uint32_t)v & 0xfffffu, hi = (uint32_t)(v >> 20);
  HEART_HALF_REDUCE(uint32_t, lo, HEART_OP_ADD);
  HEART_HALF_REDUCE(uint32_t, hi, HEART_OP_ADD);
  return ((unsigned long long)hi << 20) + lo;
}
__device__ __forceinline__ uint32_t half_max_u32(uint32_t v) {
  HEART_HALF_REDUCE(uint32_t, v, HEART_OP_UMAX);
  return v;
}
__device__ __forceinline__ float half_max_f32(float v) {
  HEART_HALF_REDUCE(float, v, HEART_OP_FMAX);
  return v;
}
__device__ __forceinline__ float half_sum_f32(float v) {
  HEART_HALF_REDUCE(float, v, HEART_OP_ADD);
  return v;
}
__device__ __forceinline__ float wave_max_f32(float v) {
  HEART_WAVE_REDUCE(float, v, HEART_OP_FMAX);
  return v;
}
__device__ __forceinline__ float wave_sum_f32(float v) {
  HEART_WAVE_REDUCE(float, v, HEART_OP_ADD);
  return v;
}

// Index of the current device, for per-device caches of launch attributes (-1 on error).
constexpr int kMaxDevices = 64;
inline int current_device() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return -1;
  return dev;
}

// Per-device "done" flags for set-up that is per function and device (launch attributes,
// device queries).  Host threads may race on the first call: the set-up calls are
// idempotent and the flags are atomic, so the worst case is that two threads both do it.
struct DeviceFlags {
  std::atomic<int> v[kMaxDevices];
};
inline hipError_t set_max_lds_once(DeviceFlags &f, int dev, const void *kern, int bytes) {
  if (f.v[dev].load(std::memory_order_acquire)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) f.v[dev].store(1, std::memory_order_release);
  return e;
}
// Number of compute units of device `dev` (0 on error), queried once per device.
inline int cu_count(int dev) {
  static DeviceFlags n;
  int v = n.v[dev].load(std::memory_order_acquire);
  if (v > 0) return v;
  if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
    return 0;
  n.v[dev].store(v, std::memory_order_release);
  return v;
}

// launchers implemented per kernel file
int launch_pool(const heart_shape &s, const void *q, const void *k, float *qblk, float *kblk,
                float *qmean, float *kmean, hipStream_t st);
int launch_pool_drift(const heart_shape &s, const void *q, const void *k, float *qblk, float *kblk,
                      float *qmean, float *kmean, float *qanchor, float *kanchor,
                      unsigned char *has_anchor, const float *delta, float gate_lo, float gate_hi,
                      int commit, float *drift, unsigned char *refresh, unsigned *tickets,
                      hipStream_t st);
int launch_drift(int B, int H, int D, const float *qmean, const float *kmean, float *qanchor,
                 float *kanchor, unsigned char *has_anchor, const float *delta, float gate_lo,
                 float gate_hi, int commit, float *drift, unsigned char *refresh,
                 hipStream_t st);
int launch_mask_topp(int B, int H, int Nb, int D, const float *qblk, const float *kblk,
                     const float *scores_in, const float *tau, const unsigned char *refresh,
                     int n_always_kv, int n_dense_q, int min_keep, unsigned char *mask,
                     int *kept_idx, int *kept_count, float *scores_out, void *workspace,
                     hipStream_t st);
size_t mask_topp_workspace_bytes(int B, int H, int Nb, int D);
int launch_attn(const heart_shape &s, const void *q, const void *k, const void *v,
                const int *kept_idx, const int *kept_count, float scale, unsigned flags, void *out,
                float *lse, int *order, size_t order_bytes, hipStream_t st);

// Launch plan of heart_block_sparse_attn (attn_plan.hip).  Layout (ints): [0,8) cursors, [8,16)
// items per XCD list, [16,24) offset of each XCD's heads in the head table, [24, 24+BH) head table
// (the heads of XCD 0 in the order it walks them, then those of XCD 1, ...), [24+BH, 24+2BH) total
// kept count per head, then seq[BH*Nb], head-major: seq[head*Nb + p] = the head's p-th item,
// longest kept lists first (item = head * Nb + query block); then, in a workspace that has room
// for it, a second such sequence with the items in batches of similar kept lists.
constexpr int kNumXcd = 8;
constexpr int kPlanHdr = 24;
inline size_t attn_plan_bytes(long long BH, long long Nb) { return (kPlanHdr + (size_t)BH * ((size_t)Nb + 2)) * sizeof(int); }
// rows per head for which the second sequence exists (0 bytes otherwise)
constexpr int kNearMinRows = 64, kNearMaxRows = 1024;
inline size_t attn_near_bytes(long long BH, long long Nb) {
  return Nb >= kNearMinRows && Nb <= kNearMaxRows ? (size_t)BH * (size_t)Nb * sizeof(int) : 0;
}
// In a workspace that has room for them the cursors in use are a second set behind all that, one per
// 256 bytes (those of the header then say that every list is handed out).  Atomics on one cache line
// are served one after another, about 40 ns each whatever XCD they come from: with the eight cursors
// side by side, 1000 workgroups that ended their first rows together waited 40 us for the second
// (B = 1, 20 heads of 101 rows, one kept block a row, D = 64, block 64: 59 -> 28 us; 30 kept blocks:
// 130 -> 103 us; D = 128, block 128: 88 -> 55 and 516 -> 497 us).  Only where there can be more items
// than workgroups (512 of them at block 128, the fewest).
constexpr size_t kCursorLine = 256;
constexpr int kCursorSpread = (int)(kCursorLine / sizeof(int));
constexpr size_t kCursorBytes = (kNumXcd + 1) * kCursorLine;  // (the workspace is aligned to 16 bytes only)
constexpr long long kCursorMinItems = 512;
// A plan with everything that can go with it.  Never as much as the parts of split rows take (below), so a
// workspace of this size always holds a plan.
inline size_t attn_full_plan_bytes(long long BH, long long Nb) {
  return attn_plan_bytes(BH, Nb) + attn_near_bytes(BH, Nb) + (BH > kCursorMinItems / Nb ? kCursorBytes : 0);
}
// Workgroups, of n_wg, that work.  Four workgroups to a CU (D = 128, block 64) are faster than two where rows are many or
// keep most blocks.  Of few heads with few, uneven lists they are slower: several XCDs then share a head, more rows
// in flight find less of its K/V in the L2s, and the longest rows, slower four to a CU, decide when the launch
// ends.  So with at most kFewHeads heads and kFewRows rows, and less than kFewKept / 8 of the blocks kept, only the
// first n_few work, two to a CU (n_few = n_wg where that is no question; kept: all kept blocks).  Four -> two a CU, lists
// of the timed fields (13 to 35 % kept): one head of 844 rows 1052 -> 934 us, two 1053 -> 843, three 1218 -> 1131,
// four of 563 rows 748 -> 681 (at 3376 rows 1608 -> 1800 with stages of 64 rows, which are as fast two to a CU); random
// lists of half the blocks, one head of 520 rows 672 -> 573, two of 741 1561 -> 1569; dense lists, which keep four: one
// head of 520 rows 791 -> 1168, two of 300 460 -> 669.
constexpr int kFewHeads = 4, kFewRows = 3072, kFewKept = 5;
__host__ __device__ constexpr int working_groups(int n_wg, int n_few, long long kept, int BH, int Nb) {
  return n_few < n_wg && 8 * kept < (long long)kFewKept * BH * Nb * Nb ? n_few : n_wg;
}
// Workgroups, of n_wg, that start with an item of `list`: those of its XCD (they are dealt to the XCDs in turn); of
// one head only list 0 has items, and all of them do, in order.  The rows with the longest lists come first, and
// with the others coming for items later they would all start on XCD 0 (D = 128, block 128, lists of the timed
// fields: 465 rows 1124 -> 961 us, 296 rows 488 -> 446; D = 64, block 64, 929 rows 745 -> 687).
__host__ __device__ constexpr int list_first(int n_wg, int list, int BH) {
  return BH == 1 ? (list == 0 ? n_wg : 0) : n_wg / kNumXcd + (list < n_wg % kNumXcd ? 1 : 0);
}
// Enqueues the plan for a launch of n_wg attention workgroups, of which working_groups(n_wg, n_few, ..)
// work (with n_few < n_wg in order of length alone), over n_items items; *seq = the sequence that launch
// follows; *cursors = the spread cursors or null.  With *skip = 0 (device memory; null: no question) the plan has
// no items, and the launch that follows it ends at once.
int launch_attn_plan(int BH, int Nb, int n_wg, int n_few, int n_items, const int *kept_idx, const int *kept_count,
                     const int *skip, int *plan, size_t plan_bytes, const int **seq, int **cursors, hipStream_t st);

// Parts that the kept list of every row is split into, 1 = not (a function of the sizes alone), and the
// workspace bytes the parts take (instead of a plan; 0 if rows are not split).
int attn_split(long long BH, long long Nb, int D, int block);
size_t attn_split_bytes(long long BH, long long Nb, int D, int block);
// Shares that the kept blocks of all rows are dealt out in (0 = not), and the bytes their parts take.
int attn_shares(long long BH, long long Nb, int D, int block, bool dense);
size_t attn_share_bytes(long long BH, long long Nb, int D, int block, bool dense);
// What a call can use without shares, and the size that asks for them (always more, so it says which launch is meant).
inline size_t attn_any_bytes(long long BH, long long Nb, int D, int block) {
  const size_t plan = attn_full_plan_bytes(BH, Nb), parts = attn_split_bytes(BH, Nb, D, block);
  return plan > parts ? plan : parts;
}
inline size_t attn_balanced_bytes(long long BH, long long Nb, int D, int block, bool dense) {
  const size_t any = attn_any_bytes(BH, Nb, D, block), shares = attn_share_bytes(BH, Nb, D, block, dense);
  return shares == 0 ? any : shares > any ? shares : any + 16;
}

// Device address, on the current device, of the library's static launch-plan array
// (HEART_ATTN_STATIC_PLAN_BYTES bytes).
int attn_static_plan(int **ptr);

int launch_antidiag(const heart_shape &s, const void *q, const void *k, int stride,
                    const unsigned char *refresh, float *scores, float *workspace, hipStream_t st);
size_t antidiag_workspace_bytes(const heart_shape &s, int stride);

int launch_ebc_band_error(long long C, int T, int Y, int X, const float *err, const float *dense,
                          const double *w, double epsilon, double *ws, double *out,
                          hipStream_t st);
size_t ebc_workspace_bytes(long long C, int T, int Y, int X);
int ebc_select_host(int n, int k, const double *E, const double *S, double s_min, int *choice,
                    double *total_error, long long *nodes);
int launch_ubench_mfma(const void *a, const void *b, int n_wg, int iters, float *sink,
                       hipStream_t st);
int launch_ubench_copy(const void *src, void *dst, size_t bytes, hipStream_t st);
int launch_ubench_read(const void *src, size_t bytes, unsigned *sink, hipStream_t st);

}  // namespace heart
