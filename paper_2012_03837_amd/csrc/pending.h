// Partial sums that wait for a later launch (PendingSums), as a kernel sees them: added by a launch of their own
// (kernels_basic.hip) or by blocks behind a product's tiles (kernels_gemm_tile.hip), with the same bits.
#pragma once
#include "common.h"

namespace lp {

// out[j] (+)= sum_b partial[b, j].  Block = 64 columns x 16 row groups; group q adds rows q, q+16, ... in
// order (four independent loads in flight at a time) and the sixteen group sums are then added in order:
// a fixed tree, so the result does not depend on the launch.
constexpr int kReduceGroups = 16;
__device__ __forceinline__ float group_sum(const float* __restrict__ partial, int nblk, int n, int j, int q) {
  float a = 0.f;
  int b = q;
  for (; b + 3 * kReduceGroups < nblk; b += 4 * kReduceGroups) {
    float v0 = partial[(size_t)b * n + j], v1 = partial[(size_t)(b + kReduceGroups) * n + j];
    float v2 = partial[(size_t)(b + 2 * kReduceGroups) * n + j], v3 = partial[(size_t)(b + 3 * kReduceGroups) * n + j];
    a += v0; a += v1; a += v2; a += v3;
  }
  for (; b < nblk; b += kReduceGroups) a += partial[(size_t)b * n + j];
  return a;
}

// first[i]: number of the first block (of 64 columns) of sum i.
struct PendingTable { PendingSums::Sum s[kMaxPending]; int first[kMaxPending]; int count, blocks; };

// Block `block` of the table's, in a block of WAVES (4, 8 or 16) wavefronts, in the order of group_sum; sh holds kReduceGroups
// rows of 64 floats.
template <int WAVES>
__device__ __forceinline__ void add_pending_block(const PendingTable& t, int block, float (*sh)[64]) {
  int p = 0;
#pragma unroll
  for (int i = 1; i < kMaxPending; ++i)
    if (i < t.count && block >= t.first[i]) p = i;
  const float* part = t.s[p].part;
  const int n = t.s[p].n, nblk = t.s[p].nblk;
  const int lc = threadIdx.x & 63, j = (block - t.first[p]) * 64 + lc;
  constexpr int GP = kReduceGroups / WAVES;        // groups of a wave, side by side: each is a chain of memory latencies
  const int q0 = threadIdx.x >> 6;
  float a[GP];
#pragma unroll
  for (int g = 0; g < GP; ++g) a[g] = 0.f;
  if (j < n) {
    constexpr int U = GP > 1 ? 8 : 4;
    int b = 0;                                     // row b + group
    for (; b + U * kReduceGroups <= nblk; b += U * kReduceGroups) {
      float v[U][GP];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int g = 0; g < GP; ++g) v[u][g] = part[(size_t)(b + u * kReduceGroups + q0 + g * WAVES) * n + j];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int g = 0; g < GP; ++g) a[g] += v[u][g];
    }
    for (; b < nblk; b += kReduceGroups)
#pragma unroll
      for (int g = 0; g < GP; ++g) {
        const int r = b + q0 + g * WAVES;
        if (r < nblk) a[g] += part[(size_t)r * n + j];
      }
  }
#pragma unroll
  for (int g = 0; g < GP; ++g) sh[q0 + g * WAVES][lc] = a[g];
  __syncthreads();
  if (threadIdx.x < 64 && j < n) {
    float v = 0.f;
#pragma unroll
    for (int g = 0; g < kReduceGroups; ++g) v += sh[g][lc];
    float* out = t.s[p].out;
    out[j] = t.s[p].accumulate ? out[j] + v : v;
  }
}

// Takes everything that is pending.
static inline PendingTable take_pending(PendingSums* ps) {
  PendingTable t = {};
  if (!ps) return t;
  for (int i = 0; i < ps->count; ++i) {
    t.s[i] = ps->s[i];
    t.first[i] = t.blocks;
    t.blocks += (ps->s[i].n + 63) / 64;
  }
  t.count = ps->count;
  ps->count = 0; ps->used = 0;
  return t;
}

}  // namespace lp
