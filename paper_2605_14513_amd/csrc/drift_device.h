// drift_workgroup: the mean-pooled drift (Eq. 4), the reuse rule (Sec. 4.2; Alg. 1), the
// layer-level gate (thresholds from the appendix on HEART configurations) and the anchor
// update for ONE batch item, executed by one whole workgroup of any multiple of 64 lanes.
// Called by the standalone drift kernel and by the tail of the fused pooling kernel.
#pragma once

#include "heart_internal.h"

namespace heart {

constexpr int kDriftHeadsPerPass = 4;

// Where the token means of a batch item (offset o = h * D + d) come from; the values and the arithmetic are the same.
struct DriftMeans {  // written before this launch, or by this workgroup
  const float *q, *k;
  __device__ __forceinline__ float qm(size_t o) const { return q[o]; }
  __device__ __forceinline__ float km(size_t o) const { return k[o]; }
};
struct DriftMeansAcross {  // written by other workgroups of this launch, possibly on another XCD
  const float *q, *k;
  __device__ __forceinline__ float qm(size_t o) const { return __hip_atomic_load(q + o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ float km(size_t o) const { return __hip_atomic_load(k + o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// What the stage reads of a wavefront's heads h0 .. h0 + kDriftHeadsPerPass - 1 that no other workgroup of the launch writes
// before the stage is over (of heads past the last: the last one's, which is computed and not stored).  All loads are issued
// unconditionally (the anchor buffers always exist); a head without an anchor ignores the value.
template <int kSlots>
struct DriftAnchors {
  float q[kDriftHeadsPerPass][kSlots], k[kDriftHeadsPerPass][kSlots], delta[kDriftHeadsPerPass];
  bool has[kDriftHeadsPerPass];
  __device__ __forceinline__ void load_head(int u, int b, int h0, int H, int D, const float *qanchor, const float *kanchor,
                                            const unsigned char *has_anchor, const float *dl) {
    const int lane = threadIdx.x & 63, h = min(h0 + u, H - 1);
    const size_t o = ((size_t)b * H + h) * D;
    has[u] = has_anchor[(size_t)b * H + h] != 0;
    delta[u] = dl[h];
#pragma unroll
    for (int c = 0; c < kSlots; ++c) {
      const int d = lane + 64 * c;
      q[u][c] = d < D ? qanchor[o + d] : 0.f;
      k[u][c] = d < D ? kanchor[o + d] : 0.f;
    }
  }
  __device__ __forceinline__ void load(int b, int h0, int H, int D, const float *qanchor, const float *kanchor,
                                       const unsigned char *has_anchor, const float *dl) {
#pragma unroll
    for (int u = 0; u < kDriftHeadsPerPass; ++u) load_head(u, b, h0, H, D, qanchor, kanchor, has_anchor, dl);
  }
};

// lds: 2 H bytes of LDS (marks, then final decisions).  Every lane of the workgroup must
// call this (it contains workgroup barriers).  kSlots: elements of a lane, D / 64 or 1.  kKeep: where
// one pass takes all heads, the lanes keep the means that they compared, and the anchors are written from
// registers instead of after a second pass of loads.  kLoaded: anchors holds those of heads 4 * wavefront on already.
// (Loaded ahead where nothing is done meanwhile, and with room for the largest D in every lane, they only cost
// registers, 67 -> 128 and 24 bytes of scratch a lane: heart_drift of 40 heads of 128 5.9 -> 7.7 us, 5.6 like this.)
template <int kSlots, bool kKeep, bool kLoaded, class Means>
__device__ __forceinline__ void drift_workgroup(
    int b, int H, int D, const Means &mean, DriftAnchors<kSlots> &anchors, float *qanchor, float *kanchor,
    unsigned char *has_anchor, const float *delta, float gate_lo, float gate_hi, int commit,
    float *drift, unsigned char *refresh, unsigned char *lds) {
  unsigned char *mark = lds;     // [H]: bit 0 the mark, bit 1 an anchor is there
  unsigned char *fin = lds + H;  // [H]
  __shared__ int n_mark_sh;

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int n_waves = blockDim.x >> 6;
  constexpr int kKept = kKeep ? kSlots : 1;
  const bool keep = kKeep && H <= n_waves * kDriftHeadsPerPass;
  float kept_q[kDriftHeadsPerPass][kKept], kept_k[kDriftHeadsPerPass][kKept];
  const size_t item = (size_t)b * H * D;

  // A wavefront takes kDriftHeadsPerPass heads at a time and issues the loads of all of them
  // before it reduces any: the stage is bound by dependent memory round trips, not by bandwidth.
  for (int h0 = wave * kDriftHeadsPerPass; h0 < H; h0 += n_waves * kDriftHeadsPerPass) {
    if (kLoaded && h0 >= n_waves * kDriftHeadsPerPass) anchors.load(b, h0, H, D, qanchor, kanchor, has_anchor, delta);
    float a[kDriftHeadsPerPass][kSlots];
#pragma unroll
    for (int u = 0; u < kDriftHeadsPerPass; ++u) {
      const size_t o = (size_t)min(h0 + u, H - 1) * D;
      if (!kLoaded) anchors.load_head(u, b, h0, H, D, qanchor, kanchor, has_anchor, delta);
#pragma unroll
      for (int c = 0; c < kSlots; ++c) {
        a[u][c] = 0.f;
        const int d = lane + 64 * c;
        if (d < D) {
          const float qv = mean.qm(o + d), kv = mean.km(o + d);
          const float dq = fabsf(anchors.q[u][c] - qv);
          const float dk = fabsf(anchors.k[u][c] - kv);
          a[u][c] = dq + dk;
          if (kKeep) kept_q[u][c < kKept ? c : 0] = qv, kept_k[u][c < kKept ? c : 0] = kv;
        }
      }
    }
#pragma unroll
    for (int u = 0; u < kDriftHeadsPerPass; ++u) {
      const int h = h0 + u;
      // steps with s >= 64: a[i] += a[i+s]  <=>  slot c += slot c + s/64
#pragma unroll
      for (int s = kSlots / 2; s >= 1; s >>= 1)
#pragma unroll
        for (int c = 0; c < kSlots / 2; ++c)
          if (c < s) a[u][c] = a[u][c] + a[u][c + s];
      float v = a[u][0];
      // steps with s < 64 (lanes >= D hold +0, adding it is exact)
#pragma unroll
      for (int s = 32; s >= 1; s >>= 1) {
        float o2 = __shfl_xor(v, s, 64);
        if (s < D) v = v + o2;
      }
      if (lane == 0 && h < H) {
        float dv = anchors.has[u] ? v : __builtin_inff();
        drift[(size_t)b * H + h] = dv;
        mark[h] = ((!anchors.has[u] || dv > anchors.delta[u]) ? 1 : 0) | (anchors.has[u] ? 2 : 0);
      }
    }
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t n = 0;
    for (int h = lane; h < H; h += 64) n += mark[h] & 1;
    n = wave_sum_u32(n);
    if (lane == 0) n_mark_sh = (int)n;
  }
  __syncthreads();
  const float frac = __fdiv_rn((float)n_mark_sh, (float)H);
  for (int h = threadIdx.x; h < H; h += blockDim.x) {
    unsigned char r;
    if (frac < gate_lo)
      r = mark[h] & 2 ? 0 : 1;
    else if (frac > gate_hi)
      r = 1;
    else
      r = mark[h] & 1;
    fin[h] = r;
    refresh[(size_t)b * H + h] = r;
  }
  __syncthreads();
  if (commit && keep) {
#pragma unroll
    for (int u = 0; u < kDriftHeadsPerPass; ++u) {
      const int h = wave * kDriftHeadsPerPass + u;
      if (h < H && fin[h]) {
#pragma unroll
        for (int c = 0; c < kKept; ++c) {
          qanchor[item + (size_t)h * D + lane + 64 * c] = kept_q[u][c];
          kanchor[item + (size_t)h * D + lane + 64 * c] = kept_k[u][c];
        }
      }
    }
  } else if (commit) {
    // (a lane loads its elements of a batch of passes before it stores any: the loads are
    // independent round trips, the stores conditional on the head's decision)
    constexpr int kBatch = 4;
    const int n = H * D;
    for (int e0 = threadIdx.x; e0 < n; e0 += kBatch * blockDim.x) {
      float qv[kBatch], kv[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int e = min(e0 + u * (int)blockDim.x, n - 1);
        qv[u] = mean.qm(e);
        kv[u] = mean.km(e);
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int e = e0 + u * (int)blockDim.x;
        if (e < n && fin[e / D]) {
          qanchor[item + e] = qv[u];
          kanchor[item + e] = kv[u];
        }
      }
    }
  }
  if (commit)
    for (int h = threadIdx.x; h < H; h += blockDim.x)
      if (fin[h]) has_anchor[(size_t)b * H + h] = 1;
}

}  // namespace heart
