// The log-sum-exp of a row of bf16 logits by groups of 64 columns: m_g = max z, s_g = sum exp(z - m_g), eight lanes of eight
// columns each, then s = sum_g s_g exp(m_g - m) as 32 sums over every 32nd group in order (64 over every 64th for more than 24576
// columns), added in a fixed tree.  The
// cross-entropy kernel (kernels_fast_bf16.hip) takes a row this way, and an evaluation's product (kernels_gemm_dma.hip), whose waves
// own 64 columns, leaves the groups' pairs instead of logits: the same steps, so the same bits.
#pragma once
#include "common.h"

namespace lp {

template <int CTRL>
__device__ __forceinline__ float dpp_lane(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// Over lanes 8 q .. 8 q + 7, all of them active: xor 1, xor 2, 7 - i.
__device__ __forceinline__ float max_of_8(float v) {
  v = fmaxf(v, dpp_lane<0xb1>(v));
  v = fmaxf(v, dpp_lane<0x4e>(v));
  return fmaxf(v, dpp_lane<0x141>(v));
}
__device__ __forceinline__ float sum_of_8(float v) {
  v += dpp_lane<0xb1>(v);
  v += dpp_lane<0x4e>(v);
  return v + dpp_lane<0x141>(v);
}
// A group's pair in all its eight lanes, z this lane's columns (-inf where there is none).  A group of -inf has the sum 0.
__device__ __forceinline__ void group_stats(const float (&z)[8], float& m, float& s) {
  m = z[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) m = fmaxf(m, z[e]);
  m = max_of_8(m);
  const float ref = m == -INFINITY ? 0.f : m;
  s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) s += __expf(z[e] - ref);
  s = sum_of_8(s);
}

// What the product of a head's logits leaves where only the loss is wanted: pair[row * groups + column / 64], and the label's
// logit of each row (not written where the label is outside [0, n)).
struct GroupStats { float2* pair; float* zy; const int32_t* y; int groups; };

}  // namespace lp
