// Arithmetic of the block scores: a 512-byte summary lies over the 32 lanes of a half-wavefront (lanes 0-15 hold 8 channels
// of kmin each, lanes 16-31 of kmax), the products are summed over them by a butterfly.  Shared by the score kernel and by
// the selection of short sequences, which scores its blocks itself.
#pragma once

#include "dsk_attn_fold.hpp"
#include "dsk_common.hpp"

namespace dsk {

// value of lane (lane ^ M) of the same half-wave: on the vector ALU's data-parallel path for
// M < 16 (quad permutes and row mirrors; a mirror of 8 followed by a reversal inside quads flips
// lane bit 2, a mirror of 16 followed by a mirror of 8 flips bit 3), through the LDS crossbar for 16
constexpr int kDppQuadReverse = 0x1B;  // quad_perm [3,2,1,0]
template <int M>
__device__ __forceinline__ float xchg_half_wave(float v) {
  if constexpr (M == 1) return dpp_f<kDppSwap1>(v);
  else if constexpr (M == 2) return dpp_f<kDppSwap2>(v);
  else if constexpr (M == 4) return dpp_f<kDppQuadReverse>(dpp_f<kDppHalfMirror>(v));
  else if constexpr (M == 8) return dpp_f<kDppHalfMirror>(dpp_f<kDppMirror>(v));
  else return shfl_xor_f(v, M);
}

// Sum V (a power of two, <= 32) per-lane values over the 32 lanes of a half-wave.  While more
// than one value is left, a step over lane bit M halves them: the lane keeps the upper half of
// the value indices if its bit M is set (the lower half otherwise) and adds what its partner
// (lane ^ M) carried for that half; afterwards plain exchanges finish the sum.  Steps run from
// lane bit 0 upwards, so that the steps with many values to exchange are the cheap ones.  On
// return v[0] is the finished sum of original value index `idx` (built MSB-first from the lane
// bits of the halving steps, i.e. from the low log2(V) lane bits, bit 0 first).
template <int N, int V, int M>
__device__ __forceinline__ void half_wave_reduce(float (&v)[N], int lane, int& idx) {
  if constexpr (M <= 16) {
    if constexpr (V >= 2) {
      const bool up = (lane & M) != 0;
#pragma unroll
      for (int x = 0; x < V / 2; ++x) {
        const float send = up ? v[x] : v[x + V / 2];
        const float keep = up ? v[x + V / 2] : v[x];
        v[x] = keep + xchg_half_wave<M>(send);
      }
      idx = idx * 2 + (up ? 1 : 0);
      half_wave_reduce<N, V / 2, M * 2>(v, lane, idx);
    } else {
      v[0] += xchg_half_wave<M>(v[0]);
      half_wave_reduce<N, 1, M * 2>(v, lane, idx);
    }
  }
}

// dot product of the 8 channels of a summary (widened) with the q+ or q- of a head, in channel order
__device__ __forceinline__ float dot8_f32(const float (&q)[8], const float (&k)[8]) {
  float acc = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) acc = fmaf(q[i], k[i], acc);
  return acc;
}

// q+ (lanes holding kmax) or q- (lanes holding kmin) of 8 channels as packed bf16 pairs: the halves whose sign does not fit
// are zeroed, both are exact in bf16
__device__ __forceinline__ void keep_sign(const uint4& q, bool is_max, uint32_t (&out)[4]) {
  const uint32_t wds[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t neg = ((uint32_t)((int32_t)(wds[k] << 16) >> 31) & 0xFFFFu) |
                         ((uint32_t)((int32_t)wds[k] >> 31) & 0xFFFF0000u);   // ones over negative halves
    out[k] = wds[k] & (is_max ? ~neg : neg);
  }
}

// this lane's part of the scores of N blocks for one query head.  FP32: single-precision multiply-adds in channel order
// (group widths that are no power of two up to 8) instead of the packed bf16 dot instruction.
template <int N, bool FP32>
__device__ __forceinline__ void score_parts(const uint4 (&kv)[N], const uint4& q, bool is_max, float (&v)[N]) {
  if constexpr (FP32) {
    float qs[8];
    unpack8(q, qs);
#pragma unroll
    for (int k = 0; k < 8; ++k) qs[k] = is_max ? fmaxf(qs[k], 0.0f) : fminf(qs[k], 0.0f);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      float f[8];
      unpack8(kv[u], f);
      v[u] = dot8_f32(qs, f);
    }
  } else {
    uint32_t qp[4];
    keep_sign(q, is_max, qp);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      float acc = dot2_bf16(qp[0], kv[u].x, 0.0f);
      acc = dot2_bf16(qp[1], kv[u].y, acc);
      acc = dot2_bf16(qp[2], kv[u].z, acc);
      v[u] = dot2_bf16(qp[3], kv[u].w, acc);
    }
  }
}

}  // namespace dsk
