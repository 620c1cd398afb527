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

// q+ (lanes holding kmax) or q- (lanes holding kmin) of 8 channels as packed bf16 pairs: the halves whose sign does not fit
// are zeroed, both are exact in bf16 (a NaN stays in one of them)
__device__ __forceinline__ void keep_sign(const uint4& q, bool is_max, uint32_t (&out)[4]) {
  const uint32_t wds[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t neg = ((uint32_t)((int32_t)(wds[k] << 16) >> 31) & 0xFFFFu) |
                         ((uint32_t)((int32_t)wds[k] >> 31) & 0xFFFF0000u);   // ones over negative halves
    out[k] = wds[k] & (is_max ? ~neg : neg);
  }
}

// this lane's part of the score of a block: 8 channels of its summary with keep_sign's q, on the packed bf16 dot instruction,
// neither operand widened.  (Groups whose width is no power of two up to 8 had single-precision multiply-adds in channel order,
// 16 instructions more a block and head and as far from 64 bits, 3.3e-8 to 4.4e-8 of the norm: decode steps of 40 / 8 heads 44.3
// -> 41.8 us at three sequences of 107K tokens, 24.1 -> 22.9 at four of 7K; 28 / 4, shared lists, eight of 50K 42.0 -> 39.2.)
__device__ __forceinline__ float score_part(const uint32_t (&qp)[4], const uint4& k) {
  float acc = dot2_bf16(qp[0], k.x, 0.0f);
  acc = dot2_bf16(qp[1], k.y, acc);
  acc = dot2_bf16(qp[2], k.z, acc);
  return dot2_bf16(qp[3], k.w, acc);
}

}  // namespace dsk
