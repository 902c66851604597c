// A small classifier head on [rows, in] features (at most 32 classes, 1024 features): logits, cross-entropy, dZ and
// the gradient of the features in one kernel, one wave per row.  As separate launches (product, softmax, product) each
// is a memory latency and a launch gap long and nothing else: 128 x 10 x 256 fp32 took 6 + 3.4 + 12 us and their gaps,
// 256 x 10 x 512 bf16 9.3 + 4.7 + 6 us; 4.5 and 5.5 us here.  The weights (at most 128 KB) are read from L2 by every
// wave, which is why the class count is limited.
// Logits are rounded to the compute dtype before the softmax, and dZ is stored in it for the weight gradient.
#include "common.h"

namespace lp {

namespace {

__device__ __forceinline__ float wsum64(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wmax64(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

template <typename T, int NI>
__global__ void __launch_bounds__(256) k_head_ce(const T* __restrict__ feat, const T* __restrict__ w, const float* __restrict__ bias,
                                                 const int32_t* __restrict__ y, float* __restrict__ loss_rows, T* __restrict__ dz,
                                                 T* __restrict__ dfeat, int rows, int in, int ncls, int backward, float inv_rows) {
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= rows) return;
  float h[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int k = lane + 64 * i;
    h[i] = k < in ? to_f(feat[(size_t)row * in + k]) : 0.f;
  }
  const int yy = y[row];
  float z = -INFINITY;             // lane c holds the logit of class c
  constexpr int U = NI >= 16 ? 2 : 4;      // classes with their loads in flight together
  for (int c0 = 0; c0 < ncls; c0 += U) {
    float s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const T* wr = w + (size_t)(c0 + u < ncls ? c0 + u : ncls - 1) * in;
      s[u] = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int k = lane + 64 * i;
        s[u] = fmaf(h[i], to_f(wr[k < in ? k : in - 1]), s[u]);      // h is zero past the end
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float t = wsum64(s[u]);
      if (lane == c0 + u) z = t;
    }
  }
  if (lane < ncls) z = to_f(from_f<T>(bias ? z + bias[lane] : z));
  else z = -INFINITY;
  const float m = wmax64(z);
  const float lse = m + __logf(wsum64(lane < ncls ? __expf(z - m) : 0.f));
  const bool y_ok = yy >= 0 && yy < ncls;      // a label outside [0, ncls) contributes lse and no one-hot term
  const float zy = __shfl(z, y_ok ? yy : 0, 64);
  if (lane == 0) loss_rows[row] = lse - (y_ok ? zy : 0.f);
  if (!backward) return;
  float d = lane < ncls ? __expf(z - lse) : 0.f;
  if (lane == yy) d -= 1.f;
  const T dt = from_f<T>(d * inv_rows);
  if (lane < ncls) dz[(size_t)row * ncls + lane] = dt;
  const float dv = to_f(dt);
  float g[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) g[i] = 0.f;
  for (int c = 0; c < ncls; ++c) {
    const float dc = __shfl(dv, c, 64);
    const T* wr = w + (size_t)c * in;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int k = lane + 64 * i;
      g[i] = fmaf(dc, to_f(wr[k < in ? k : in - 1]), g[i]);
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int k = lane + 64 * i;
    if (k < in) dfeat[(size_t)row * in + k] = from_f<T>(g[i]);
  }
}

template <typename T>
hipError_t head_ce_t(const OpCtx& c, const void* feat, const void* w, const float* bias, const int32_t* y, float* loss_rows,
                     void* dz, void* dfeat, int rows, int in, int ncls, int backward, float inv_rows) {
  const int blocks = (rows + 3) / 4;
#define LP_HEAD(NI) k_head_ce<T, NI><<<blocks, 256, 0, c.stream>>>((const T*)feat, (const T*)w, bias, y, loss_rows, (T*)dz, \
                                                                   (T*)dfeat, rows, in, ncls, backward, inv_rows)
  if (in <= 128) LP_HEAD(2);
  else if (in <= 256) LP_HEAD(4);
  else if (in <= 512) LP_HEAD(8);
  else LP_HEAD(16);
#undef LP_HEAD
  return hipGetLastError();
}

}  // namespace

bool head_ce_ok(int in, int ncls) { return ncls <= 32 && in <= 1024; }
hipError_t op_head_ce(const OpCtx& c, const void* feat, const void* w, const float* bias, const int32_t* y, float* loss_rows,
                      void* dz, void* dfeat, int rows, int in, int ncls, int backward, float inv_rows) {
  ProfScope prof_(c, KC_SOFTMAX_CE);
  if (rows == 0) return hipSuccess;
  return c.dt == BF16 ? head_ce_t<bf16_t>(c, feat, w, bias, y, loss_rows, dz, dfeat, rows, in, ncls, backward, inv_rows)
                      : head_ce_t<float>(c, feat, w, bias, y, loss_rows, dz, dfeat, rows, in, ncls, backward, inv_rows);
}

}  // namespace lp
