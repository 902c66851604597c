// Small classifier heads on [rows, in] features (at most 32 classes, 1024 features): logits, cross-entropy, dZ and the
// gradient of the features in one kernel, one wave per row, up to eight heads (blocks of the network) per launch.  As
// separate launches (product, softmax, product) each is a memory latency and a launch gap long and nothing else:
// 128 x 10 x 256 fp32 took 6 + 3.4 + 12 us and their gaps, 256 x 10 x 512 bf16 9.3 + 4.7 + 6 us; 4.5 and 5.5 us here
// (four of the former in one launch: 7.3 us).
// A lane owns four consecutive features (16-byte loads), several classes' loads are in flight at a time, and the weights
// (at most 128 KB) come from L2 for every wave, which is why the class count is limited.
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
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 ld4(const bf16_t* p) {
  const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
  return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
__device__ __forceinline__ void st4(float* p, f32x4 v) { *reinterpret_cast<f32x4*>(p) = v; }
__device__ __forceinline__ void st4(bf16_t* p, f32x4 v) {
  *reinterpret_cast<bf16x4*>(p) = bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
}
// features k .. k + 3 of a row (zero past the end); VEC: rows start on, and end at, whole loads
template <bool VEC, typename T>
__device__ __forceinline__ f32x4 row4(const T* row, int k, int in) {
  if (VEC) return k < in ? ld4(row + k) : f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float v = to_f(row[k + j < in ? k + j : in - 1]);
    r[j] = k + j < in ? v : 0.f;
  }
  return r;
}

template <typename T, int NI, bool VEC>
__global__ void __launch_bounds__(256) k_head_ce(HeadTable ht, const int32_t* __restrict__ y, int rows, int backward, float inv_rows) {
  const HeadCe& H = ht.h[blockIdx.y];
  const int lane = threadIdx.x & 63, row = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= rows) return;
  const int in = H.in, ncls = H.ncls;
  const T* w = (const T*)H.w;
  const T* fr = (const T*)H.feat + (size_t)row * in;
  f32x4 h[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) h[i] = row4<VEC>(fr, 4 * lane + 256 * i, in);
  const int yy = y[row];
  float z = -INFINITY;             // lane c holds the logit of class c
  constexpr int U = 8 / NI < 2 ? 2 : 8 / NI;        // classes with their loads in flight together
  for (int c0 = 0; c0 < ncls; c0 += U) {
    f32x4 wv[U][NI];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        wv[u][i] = row4<VEC>(w + (size_t)(c0 + u < ncls ? c0 + u : ncls - 1) * in, 4 * lane + 256 * i, in);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) s = fmaf(h[i][j], wv[u][i][j], s);
      const float t = wsum64(s);
      if (lane == c0 + u) z = t;
    }
  }
  if (lane < ncls) z = to_f(from_f<T>(H.bias ? z + H.bias[lane] : z));
  else z = -INFINITY;
  const float m = wmax64(z);
  const float lse = m + __logf(wsum64(lane < ncls ? __expf(z - m) : 0.f));
  const bool y_ok = yy >= 0 && yy < ncls;      // a label outside [0, ncls) contributes lse and no one-hot term
  const float zy = __shfl(z, y_ok ? yy : 0, 64);
  if (lane == 0) H.loss_rows[row] = lse - (y_ok ? zy : 0.f);
  if (!backward) return;
  float d = lane < ncls ? __expf(z - lse) : 0.f;
  if (lane == yy) d -= 1.f;
  const T dt = from_f<T>(d * inv_rows);
  if (lane < ncls) ((T*)H.dz)[(size_t)row * ncls + lane] = dt;
  const float dv = lane < ncls ? to_f(dt) : 0.f;
  f32x4 g[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) g[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < ncls; c0 += U) {
    f32x4 wv[U][NI];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < NI; ++i)
        wv[u][i] = row4<VEC>(w + (size_t)(c0 + u < ncls ? c0 + u : ncls - 1) * in, 4 * lane + 256 * i, in);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (c0 + u >= ncls) break;                    // a zero would do, but not against an infinite weight
      const float dc = __shfl(dv, c0 + u, 64);
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) g[i][j] = fmaf(dc, wv[u][i][j], g[i][j]);
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int k = 4 * lane + 256 * i;
    const size_t o = (size_t)row * in + k;
    if (VEC) {
      if (k < in) {
        st4((T*)H.dfeat + o, g[i]);
        if (H.dfeat2) st4((T*)H.dfeat2 + o, g[i]);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (k + j < in) {
          ((T*)H.dfeat)[o + j] = from_f<T>(g[i][j]);
          if (H.dfeat2) ((T*)H.dfeat2)[o + j] = from_f<T>(g[i][j]);
        }
    }
  }
}

template <typename T, bool VEC>
hipError_t head_ce_t(const OpCtx& c, const HeadTable& ht, const int32_t* y, int rows, int backward, float inv_rows, int widest) {
  const dim3 grid((rows + 3) / 4, ht.n);
#define LP_HEAD(NI) k_head_ce<T, NI, VEC><<<grid, 256, 0, c.stream>>>(ht, y, rows, backward, inv_rows)
  if (widest <= 256) LP_HEAD(1);
  else if (widest <= 512) LP_HEAD(2);
  else if (widest <= 768) LP_HEAD(3);
  else LP_HEAD(4);
#undef LP_HEAD
  return hipGetLastError();
}

}  // namespace

bool head_ce_ok(int in, int ncls) { return ncls <= 32 && in <= 1024; }
hipError_t op_head_ce(const OpCtx& c, const HeadTable& ht, const int32_t* y, int rows, int backward, float inv_rows) {
  ProfScope prof_(c, KC_SOFTMAX_CE);
  if (rows == 0 || ht.n == 0) return hipSuccess;
  const size_t al = 4 * dtype_size(c.dt) - 1;
  bool vec = true;
  int widest = 0;
  for (int i = 0; i < ht.n; ++i) {
    const HeadCe& h = ht.h[i];
    vec = vec && h.in % 4 == 0 && (((uintptr_t)h.feat | (uintptr_t)h.w | (uintptr_t)h.dfeat | (uintptr_t)h.dfeat2) & al) == 0;
    if (h.in > widest) widest = h.in;
  }
  if (c.dt == BF16)
    return vec ? head_ce_t<bf16_t, true>(c, ht, y, rows, backward, inv_rows, widest) : head_ce_t<bf16_t, false>(c, ht, y, rows, backward, inv_rows, widest);
  return vec ? head_ce_t<float, true>(c, ht, y, rows, backward, inv_rows, widest) : head_ce_t<float, false>(c, ht, y, rows, backward, inv_rows, widest);
}

}  // namespace lp
