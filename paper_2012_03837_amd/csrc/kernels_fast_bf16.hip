// Vectorised bf16 forms of the HBM-bound kernels: one global read and one global write per element,
// 16 bytes per lane, all intermediate values in registers.
//   LayerNorm forward / backward : rows of up to 1024 elements, one wavefront per row
//   softmax cross-entropy        : rows of up to 32768 logits, a block of 256 or 512 threads per row
// Shapes outside these limits (or unaligned) use the generic kernels.
#include <type_traits>
#include "common.h"
#include "row_loss.h"

namespace lp {

namespace {

__device__ __forceinline__ float wsum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wmax(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ void load8(const bf16_t* p, float* v) {
  bf16x8 t = *reinterpret_cast<const bf16x8*>(p);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)t[e];
}
__device__ __forceinline__ void store8(bf16_t* p, const float* v) {
  bf16x8 t;
#pragma unroll
  for (int e = 0; e < 8; ++e) t[e] = (bf16_t)v[e];
  *reinterpret_cast<bf16x8*>(p) = t;
}
__device__ __forceinline__ void loadf8(const float* p, float* v) {
  f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
}

constexpr float kEps = 1e-5f;

template <int NCH>
__global__ void __launch_bounds__(256) k_ln_fwd_v(const bf16_t* __restrict__ x, const float* __restrict__ g,
                                                  const float* __restrict__ b, bf16_t* __restrict__ y,
                                                  float* __restrict__ mean, float* __restrict__ rstd, int rows, int d) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int nch = d >> 3;
  const bf16_t* xr = x + (size_t)row * d;
  float v[NCH][8];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    int c = lane + 64 * i;
    if (c < nch) {
      load8(xr + 8 * c, v[i]);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += v[i][e];
    }
  }
  const float mu = wsum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (lane + 64 * i < nch) {
#pragma unroll
      for (int e = 0; e < 8; ++e) { float t = v[i][e] - mu; q += t * t; }
    }
  const float rs = rsqrtf(wsum(q) / (float)d + kEps);
  bf16_t* yr = y + (size_t)row * d;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    int c = lane + 64 * i;
    if (c < nch) {
      float gg[8], bb[8], o[8];
      loadf8(g + 8 * c, gg); loadf8(b + 8 * c, bb);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (v[i][e] - mu) * rs * gg[e] + bb[e];
      store8(yr + 8 * c, o);
    }
  }
  if (lane == 0) { mean[row] = mu; rstd[row] = rs; }
}

constexpr int kRowsPerBlock = kLnFastRows;
// Backward; block partials of dg and db go to partial[blk][d] and partial[nblk + blk][d].  A wave owns four
// rows of its block's sixteen and keeps the next row's loads (x, dy and the addend, 16 bytes per lane each) in
// flight while it reduces and writes the current one: with one row at a time the kernel is a chain of memory
// latencies, not a stream.
template <int NCH>
__global__ void __launch_bounds__(256) k_ln_bwd_v(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ x,
                                                  const float* __restrict__ mean, const float* __restrict__ rstd,
                                                  const float* __restrict__ g, const bf16_t* __restrict__ add,
                                                  bf16_t* __restrict__ dx, float* __restrict__ partial, int rows,
                                                  int d) {
  extern __shared__ float sh[];   // [4 waves][2][d]
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int nch = d >> 3;
  float gg[NCH][8], pg[NCH][8], pb[NCH][8];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    int c = lane + 64 * i;
#pragma unroll
    for (int e = 0; e < 8; ++e) { pg[i][e] = 0.f; pb[i][e] = 0.f; gg[i][e] = 0.f; }
    if (c < nch) loadf8(g + 8 * c, gg[i]);
  }
  const int row0 = blockIdx.x * kRowsPerBlock;
  const float invd = 1.f / (float)d;
  constexpr int RPW = kRowsPerBlock / 4;
  bf16x8 xr[2][NCH], dr[2][NCH], ar[2][NCH];
  float mu[2], rs[2];
  auto fetch = [&](int slot, int row) {
    if (row >= rows) return;
    mu[slot] = mean[row]; rs[slot] = rstd[row];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const int c = lane + 64 * i;
      if (c < nch) {
        xr[slot][i] = *reinterpret_cast<const bf16x8*>(x + (size_t)row * d + 8 * c);
        dr[slot][i] = *reinterpret_cast<const bf16x8*>(dy + (size_t)row * d + 8 * c);
        if (add && dx) ar[slot][i] = *reinterpret_cast<const bf16x8*>(add + (size_t)row * d + 8 * c);
      }
    }
  };
  fetch(0, row0 + w);
#pragma unroll
  for (int it = 0; it < RPW; ++it) {
    const int row = row0 + w + 4 * it, cur = it & 1;
    if (row >= rows) break;
    if (it + 1 < RPW) fetch(cur ^ 1, row + 4);
    float xh[NCH][8], dxh[NCH][8];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      if (lane + 64 * i < nch) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float dv = (float)dr[cur][i][e];
          xh[i][e] = ((float)xr[cur][i][e] - mu[cur]) * rs[cur];
          dxh[i][e] = dv * gg[i][e];
          s1 += dxh[i][e];
          s2 += dxh[i][e] * xh[i][e];
          pg[i][e] += dv * xh[i][e];
          pb[i][e] += dv;
        }
      }
    }
    s1 = wsum(s1) * invd;
    s2 = wsum(s2) * invd;
    if (dx) {
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        int c = lane + 64 * i;
        if (c < nch) {
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (dxh[i][e] - s1 - xh[i][e] * s2) * rs[cur];
          if (add) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += (float)ar[cur][i][e];
          }
          store8(dx + (size_t)row * d + 8 * c, o);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    int c = lane + 64 * i;
    if (c < nch) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sh[(size_t)(w * 2) * d + 8 * c + e] = pg[i][e];
        sh[(size_t)(w * 2 + 1) * d + 8 * c + e] = pb[i][e];
      }
    }
  }
  __syncthreads();
  const int nblk = gridDim.x;
  for (int j = threadIdx.x; j < d; j += 256) {
    float a = 0.f, bsum = 0.f;
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) { a += sh[(size_t)(ww * 2) * d + j]; bsum += sh[(size_t)(ww * 2 + 1) * d + j]; }
    partial[(size_t)blockIdx.x * d + j] = a;
    partial[(size_t)(nblk + blockIdx.x) * d + j] = bsum;
  }
}

// Softmax cross-entropy with the whole row in registers (4 to 12 chunks of 8 logits per thread).  TAIL: n is not a
// multiple of 8; the last chunk reaches into the row's padding, whose values count as -inf.  Chunks from n up to
// pad_to are cleared together with the gradient's write (a padded dZ is read whole by the products behind it).
// CH: chunks of a thread that there is room for, T threads.  Room for 8192 logits where a row has no more lets three times as
// many rows into a compute unit as room for 32768 (8192 x 8000 53 -> 48 us, 2048 x 16000 29.4 -> 27.7; 8192 x 17000 103 us, 108 with 512 threads); rows of
// more than 24576 take 512 threads (8192 x 32000 194 -> 187 us).
constexpr int kCeMax = 32768;
constexpr int ce_threads(int n) { return n <= 24576 ? 256 : 512; }
template <bool TAIL, int CH, int T>
__global__ void __launch_bounds__(T) k_softmax_ce_reg(bf16_t* __restrict__ z, int64_t ld, const int32_t* __restrict__ y,
                                                      float* __restrict__ loss_rows, int n, int write_grad,
                                                      float inv_rows, int pad_to) {
  constexpr int W = T / 64;
  __shared__ float sh[2 * W];
  const int row = blockIdx.x, nch = TAIL ? (n + 7) >> 3 : n >> 3;
  bf16_t* zr = z + (size_t)row * ld;
  bf16x8 v[CH];
  float gm[CH], gs[CH];      // of the group that this thread's chunk i is an eighth of
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    int c = threadIdx.x + T * i;
    if (c < nch) {
      v[i] = __builtin_nontemporal_load(reinterpret_cast<const bf16x8*>(zr + 8 * c));
      if (TAIL) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (8 * c + e >= n) v[i][e] = (bf16_t)(-INFINITY);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < CH; ++i)
    if (T * i < nch) {
      float z8[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) z8[e] = (int)threadIdx.x + T * i < nch ? (float)v[i][e] : -INFINITY;
      group_stats(z8, gm[i], gs[i]);
      m = fmaxf(m, gm[i]);
    }
  m = wmax(m);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < W; ++w) m = fmaxf(m, sh[w]);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < CH; ++i)
    if (T * i < nch) s += gs[i] * __expf(gm[i] - m);
#pragma unroll
  for (int o = 8; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) sh[W + (threadIdx.x >> 6)] = s;
  __syncthreads();
  s = sh[W];
#pragma unroll
  for (int w = 1; w < W; ++w) s += sh[W + w];
  const float lse = m + __logf(s);
  const int yy = y[row];
  const bool y_ok = yy >= 0 && yy < n;
  if (threadIdx.x == 0) loss_rows[row] = lse - (y_ok ? (float)zr[yy] : 0.f);
  if (!write_grad) return;
  __syncthreads();   // the label's logit has been read before anything is overwritten
#pragma unroll
  for (int i = 0; i < CH; ++i) {
    int c = threadIdx.x + T * i;
    if (c < nch) {
      bf16x8 o;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float p = __expf((float)v[i][e] - lse);
        if (8 * c + e == yy) p -= 1.f;
        o[e] = (bf16_t)(p * inv_rows);
        if (TAIL && 8 * c + e >= n) o[e] = (bf16_t)0.f;
      }
      __builtin_nontemporal_store(o, reinterpret_cast<bf16x8*>(zr + 8 * c));
    }
  }
  for (int j = 8 * nch + threadIdx.x; j < pad_to; j += T) zr[j] = (bf16_t)0.f;
}

// The rows' losses from their groups' pairs: NQ lanes a row (an eighth of the cross-entropy's threads), lane q the groups q, q + NQ, ...
template <int NQ>
__global__ void __launch_bounds__(256) k_ce_finish(GroupStats g, float* __restrict__ loss_rows, int rows, int n) {
  const int row = blockIdx.x * (256 / NQ) + threadIdx.x / NQ, q = threadIdx.x % NQ;
  if (row >= rows) return;
  constexpr int I = NQ == 32 ? 12 : 8;
  float2 p[I];
  float m = -INFINITY;
#pragma unroll
  for (int i = 0; i < I; ++i) {
    p[i] = q + NQ * i < g.groups ? g.pair[(size_t)row * g.groups + q + NQ * i] : float2{-INFINITY, 0.f};
    m = fmaxf(m, p[i].x);
  }
#pragma unroll
  for (int o = 1; o < NQ; o <<= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < I; ++i)
    if (NQ * i < g.groups) s += p[i].y * __expf(p[i].x - m);
#pragma unroll
  for (int o = 1; o < 8; o <<= 1) s += __shfl_xor(s, o, 64);
  const int first = threadIdx.x & 63 & ~(NQ - 1);
  float t = __shfl(s, first, 64);
#pragma unroll
  for (int w = 8; w < NQ; w += 8) t += __shfl(s, first + w, 64);
  const int yy = g.y[row];
  if (q == 0) loss_rows[row] = m + __logf(t) - (yy >= 0 && yy < n ? g.zy[row] : 0.f);
}

bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

bool ln_fast_ok(const OpCtx& c, const void* a, const void* b, const void* cc, const void* dd, int d) {
  return c.dt == BF16 && d % 8 == 0 && d <= 1024 && al16(a) && al16(b) && (!cc || al16(cc)) && (!dd || al16(dd));
}
hipError_t ln_fwd_fast(const OpCtx& c, const void* x, const float* g, const float* b, void* y, float* mean, float* rstd,
                       int rows, int d) {
  int blocks = (rows + 3) / 4;
  if (d <= 512) k_ln_fwd_v<1><<<blocks, 256, 0, c.stream>>>((const bf16_t*)x, g, b, (bf16_t*)y, mean, rstd, rows, d);
  else k_ln_fwd_v<2><<<blocks, 256, 0, c.stream>>>((const bf16_t*)x, g, b, (bf16_t*)y, mean, rstd, rows, d);
  return hipGetLastError();
}
// Launches the backward kernel only; the caller reduces the partials (nblk blocks of d floats, twice).
hipError_t ln_bwd_fast(const OpCtx& c, const void* dy, const void* x, const float* mean, const float* rstd,
                       const float* g, const void* add, void* dx, int rows, int d, int* nblk_out) {
  int nblk = (rows + kRowsPerBlock - 1) / kRowsPerBlock;
  *nblk_out = nblk;
  if ((size_t)nblk * d * 2 > c.partial_elems) return hipErrorInvalidValue;
  size_t shm = (size_t)8 * d * sizeof(float);
  if (d <= 512)
    k_ln_bwd_v<1><<<nblk, 256, shm, c.stream>>>((const bf16_t*)dy, (const bf16_t*)x, mean, rstd, g, (const bf16_t*)add,
                                                (bf16_t*)dx, c.partial, rows, d);
  else
    k_ln_bwd_v<2><<<nblk, 256, shm, c.stream>>>((const bf16_t*)dy, (const bf16_t*)x, mean, rstd, g, (const bf16_t*)add,
                                                (bf16_t*)dx, c.partial, rows, d);
  return hipGetLastError();
}
bool ce_fast_ok(const OpCtx& c, const void* z, int64_t ld, int n) {
  return c.dt == BF16 && ld % 8 == 0 && n <= kCeMax && al16(z);
}
hipError_t ce_finish(const OpCtx& c, const GroupStats& g, float* loss_rows, int rows, int n) {
  if (ce_threads(n) == 512) k_ce_finish<64><<<(rows + 3) / 4, 256, 0, c.stream>>>(g, loss_rows, rows, n);
  else k_ce_finish<32><<<(rows + 7) / 8, 256, 0, c.stream>>>(g, loss_rows, rows, n);
  return hipGetLastError();
}
hipError_t ce_fast(const OpCtx& c, void* z, int64_t ld, const int32_t* y, float* loss_rows, int rows, int n,
                   int write_grad, float inv_rows, int pad_to) {
#define LP_CE(CH, T)                                                                                                          \
  do {                                                                                                                        \
    if (n % 8) k_softmax_ce_reg<true, CH, T><<<rows, T, 0, c.stream>>>((bf16_t*)z, ld, y, loss_rows, n, write_grad, inv_rows, pad_to); \
    else k_softmax_ce_reg<false, CH, T><<<rows, T, 0, c.stream>>>((bf16_t*)z, ld, y, loss_rows, n, write_grad, inv_rows, pad_to);     \
  } while (0)
  if (n <= 8192) LP_CE(4, 256);
  else if (n <= 16384) LP_CE(8, 256);
  else if (ce_threads(n) == 256) LP_CE(12, 256);
  else LP_CE(8, 512);
#undef LP_CE
  return hipGetLastError();
}

}  // namespace lp

// ===================================================================================================
// BatchNorm over [rows, C] bf16 with C % 8 == 0: 16 bytes (8 channels) per lane.
//   statistics : one pass; per-channel sums of (x - p) and (x - p)^2 with the pivot p = the channel's
//                value in row 0 (a sample of the distribution, so the shifted variance formula
//                S2/n - (S1/n)^2 does not cancel), per-slab partials, ordered reduction.  Channel counts whose
//                chunks do not divide 256 (see bn_shifted): sums of x and x^2 in fp64 instead
//   apply      : y = [relu]((z - mean) * rstd * g + b (+ res))
//   backward   : per-slab partial sums of dy_eff and dy_eff * xhat, then
//                dz = g * rstd * (dy_eff - mean(dy_eff) - xhat * mean(dy_eff * xhat)), dres = dy_eff
// Block = (C/8) channel chunks x floor(256 / (C/8)) row lanes (the threads left over idle: 1 of 256 at 24 channels,
// at worst 127 at 1032); any C % 8 == 0 up to 2048.  Channel counts whose chunks do not divide 256 (24, 48, 96, ...)
// ran on the generic two-pass kernels before, whose variance is a sum of squares around the mean: with row 0 far from
// the mean the shifted formula would lose bits against that (row 0 at 300 standard deviations of 39200 rows: rstd off by
// 6e-3), sums in fp64 lose none (the square of a bf16 value is exact, 2^-53 times mean^2 / variance is below
// fp32's rounding for any bf16 column).  39200 x 24, statistics of the backward pass 156 us with two bytes per lane and
// 39 blocks, 5.2 us here.
namespace lp {
namespace {

constexpr float kBnEpsV = 1e-5f;

// MODE 0: s0 = sum (z - p), s1 = sum (z - p)^2.   MODE 1: s0 = sum dy_eff, s1 = sum dy_eff * xhat.
// MODE 2: s0 = sum z, s1 = sum z^2 in fp64, left as two floats each ([4][nslab][C]: s0, s1, what they lack).
template <int MODE>
__global__ void __launch_bounds__(256) k_bn_partial_v(const bf16_t* __restrict__ a, const bf16_t* __restrict__ yrelu,
                                                      const bf16_t* __restrict__ z, const float* __restrict__ mean,
                                                      const float* __restrict__ rstd, float* __restrict__ partial,
                                                      int rows, int C, int slab, int relu) {
  typedef typename std::conditional<MODE == 2, double, float>::type acc_t;
  extern __shared__ __attribute__((aligned(16))) char sh_bytes[];
  acc_t* sh = reinterpret_cast<acc_t*>(sh_bytes);        // [2][RL][C]
  const int cpr = C >> 3, RL = 256 / cpr;
  const int cc = threadIdx.x % cpr, rl = threadIdx.x / cpr;
  const int r0 = blockIdx.x * slab;
  const int r1 = r0 + slab < rows ? r0 + slab : rows;
  acc_t s0[8], s1[8];
  float p[8], q[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { s0[e] = 0; s1[e] = 0; }
  if (rl < RL) {
    if (MODE == 0) load8(z + 8 * cc, p);                      // pivot: row 0
    else if (MODE == 1) { loadf8(mean + 8 * cc, p); loadf8(rstd + 8 * cc, q); }
    // four rows' loads in flight per thread (twelve 16-byte loads in the backward pass)
    for (int r = r0 + rl; r < r1; r += 4 * RL) {
      bf16x8 av[4], zv[4], yv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int ru = r + u * RL < r1 ? r + u * RL : r;
        const size_t off = (size_t)ru * C + 8 * cc;
        av[u] = *reinterpret_cast<const bf16x8*>(a + off);
        if (MODE == 1) {
          zv[u] = *reinterpret_cast<const bf16x8*>(z + off);
          if (relu) yv[u] = *reinterpret_cast<const bf16x8*>(yrelu + off);
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (r + u * RL >= r1) break;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          float v = (float)av[u][e];
          if (MODE == 0) { const float t = v - p[e]; s0[e] += t; s1[e] += t * t; }
          else if (MODE == 2) { const acc_t t = v; s0[e] += t; s1[e] += t * t; }
          else {
            if (relu) v = (float)yv[u][e] > 0.f ? v : 0.f;
            s0[e] += v; s1[e] += v * ((float)zv[u][e] - p[e]) * q[e];
          }
        }
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sh[(size_t)rl * C + 8 * cc + e] = s0[e];
      sh[(size_t)(RL + rl) * C + 8 * cc + e] = s1[e];
    }
  }
  __syncthreads();
  const int nslab = gridDim.x;
  for (int j = threadIdx.x; j < C; j += 256) {
    acc_t t0 = 0, t1 = 0;
    for (int r = 0; r < RL; ++r) { t0 += sh[(size_t)r * C + j]; t1 += sh[(size_t)(RL + r) * C + j]; }
    partial[(size_t)blockIdx.x * C + j] = (float)t0;
    partial[(size_t)(nslab + blockIdx.x) * C + j] = (float)t1;
    if (MODE == 2) {          // nothing where the float is infinite already
      const acc_t l0 = t0 - (acc_t)(float)t0, l1 = t1 - (acc_t)(float)t1;
      partial[(size_t)(2 * nslab + blockIdx.x) * C + j] = __builtin_isfinite((float)t0) ? (float)l0 : 0.f;
      partial[(size_t)(3 * nslab + blockIdx.x) * C + j] = __builtin_isfinite((float)t1) ? (float)l1 : 0.f;
    }
  }
}
// Adds the slab partials in order (CW channels x 1024 / CW slab groups per block: group q adds slabs q, q + groups, ...
// with two independent pairs of loads in flight, then the group sums are added in order) and finishes.
// 64 channels a block, or 16 where the slabs are many: with 1024 slabs of 64 channels one block of 16 groups was a chain of
// sixteen memory latencies (9 us, with nothing beside it on the way from one convolution to the next).
// mode 0: forward statistics (needs the pivots from row 0 of z); with aux0 / aux1 the batch mean and unbiased
// variance are also folded into those running statistics with weight auxf.  mode 1: plain sums into out0, out1;
// with aux0 / aux1 they are also written (auxf == 0) or added (auxf != 0) there: the shift and gain gradients.
constexpr int kBnFinishThreads = 1024, kBnManySlabs = 128;
// The groups' sums added in order: sixteen one after the other, or 64 as eight times eight.
template <int CW, typename A>
__device__ __forceinline__ void bn_group_sums(A (&sh)[2][kBnFinishThreads / CW][CW], int q, int lc, A& a, A& b) {
  constexpr int G = kBnFinishThreads / CW;
  if constexpr (G == 64) {
    if (q < 8) {
      a = 0; b = 0;
#pragma unroll
      for (int g = 0; g < 8; ++g) { a += sh[0][8 * q + g][lc]; b += sh[1][8 * q + g][lc]; }
    }
    __syncthreads();
    if (q < 8) { sh[0][q][lc] = a; sh[1][q][lc] = b; }
    __syncthreads();
  }
  a = 0; b = 0;
#pragma unroll
  for (int g = 0; g < (G == 64 ? 8 : G); ++g) { a += sh[0][g][lc]; b += sh[1][g][lc]; }
}
template <int CW>
__global__ void __launch_bounds__(kBnFinishThreads)
k_bn_finish_v(const float* __restrict__ partial, int nslab, int C, int rows, const bf16_t* __restrict__ z,
              float* __restrict__ out0, float* __restrict__ out1, int mode, float* __restrict__ aux0 = nullptr,
              float* __restrict__ aux1 = nullptr, float auxf = 0.f) {
  constexpr int kBnFinishGroups = kBnFinishThreads / CW;
  __shared__ float sh[2][kBnFinishGroups][CW];
  const int lc = threadIdx.x % CW, q = threadIdx.x / CW;
  const int j = blockIdx.x * CW + lc;
  float a = 0.f, b = 0.f;
  if (j < C) {
    int s = q;
    for (; s + 3 * kBnFinishGroups < nslab; s += 4 * kBnFinishGroups) {      // eight loads in flight
      float av[4], bv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        av[u] = partial[(size_t)(s + u * kBnFinishGroups) * C + j];
        bv[u] = partial[(size_t)(nslab + s + u * kBnFinishGroups) * C + j];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { a += av[u]; b += bv[u]; }
    }
    for (; s + kBnFinishGroups < nslab; s += 2 * kBnFinishGroups) {
      const float a0 = partial[(size_t)s * C + j], b0 = partial[(size_t)(nslab + s) * C + j];
      const float a1 = partial[(size_t)(s + kBnFinishGroups) * C + j], b1 = partial[(size_t)(nslab + s + kBnFinishGroups) * C + j];
      a += a0; a += a1; b += b0; b += b1;
    }
    for (; s < nslab; s += kBnFinishGroups) { a += partial[(size_t)s * C + j]; b += partial[(size_t)(nslab + s) * C + j]; }
  }
  sh[0][q][lc] = a; sh[1][q][lc] = b;
  __syncthreads();
  bn_group_sums<CW>(sh, q, lc, a, b);
  if (q != 0 || j >= C) return;
  if (mode == 0) {
    const float inv = 1.f / (float)rows, m1 = a * inv;
    float var = b * inv - m1 * m1;
    var = var > 0.f ? var : 0.f;
    const float mu = (float)z[j] + m1;
    out0[j] = mu;
    out1[j] = rsqrtf(var + kBnEpsV);
    if (aux0) {   // running statistics take the unbiased batch variance
      const float unb = rows > 1 ? var * ((float)rows / (float)(rows - 1)) : var;
      aux0[j] = (1.f - auxf) * aux0[j] + auxf * mu;
      aux1[j] = (1.f - auxf) * aux1[j] + auxf * unb;
    }
  } else {
    out0[j] = a; out1[j] = b;
    if (aux0) {
      aux0[j] = auxf != 0.f ? aux0[j] + a : a;
      aux1[j] = auxf != 0.f ? aux1[j] + b : b;
    }
  }
}
// Forward statistics from the fp64 sums of k_bn_partial_v<2>, in the same order.  A variance of NaN (an infinity in the
// column) stays one.
template <int CW>
__global__ void __launch_bounds__(kBnFinishThreads)
k_bn_finish_wide(const float* __restrict__ partial, int nslab, int C, int rows, float* __restrict__ mean,
                 float* __restrict__ rstd, float* __restrict__ run_mean, float* __restrict__ run_var, float mom) {
  constexpr int kBnFinishGroups = kBnFinishThreads / CW;
  __shared__ double sh[2][kBnFinishGroups][CW];
  const int lc = threadIdx.x % CW, q = threadIdx.x / CW;
  const int j = blockIdx.x * CW + lc;
  double a = 0, b = 0;
  if (j < C) {
    const size_t part = (size_t)nslab * C;
    for (int s = q; s < nslab; s += 4 * kBnFinishGroups) {      // sixteen loads in flight
      float v[4][4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int su = s + u * kBnFinishGroups < nslab ? s + u * kBnFinishGroups : s;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[u][k] = partial[k * part + (size_t)su * C + j];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (s + u * kBnFinishGroups >= nslab) break;
        a += (double)v[u][0] + (double)v[u][2];
        b += (double)v[u][1] + (double)v[u][3];
      }
    }
  }
  sh[0][q][lc] = a; sh[1][q][lc] = b;
  __syncthreads();
  bn_group_sums<CW>(sh, q, lc, a, b);
  if (q != 0 || j >= C) return;
  const double m1 = a / rows, v1 = b / rows - m1 * m1;
  const float mu = (float)m1, var = v1 < 0 ? 0.f : (float)v1;
  mean[j] = mu;
  rstd[j] = rsqrtf(var + kBnEpsV);
  if (run_mean) {   // running statistics take the unbiased batch variance
    const float unb = rows > 1 ? var * ((float)rows / (float)(rows - 1)) : var;
    run_mean[j] = (1.f - mom) * run_mean[j] + mom * mu;
    run_var[j] = (1.f - mom) * run_var[j] + mom * unb;
  }
}
// Forward statistics from the per-slab sums the convolution kernel left (ConvStats: slab t has its own pivot p_t, the
// first of its slab_rows rows): every slab is shifted to slab 0's pivot P, with d = p_t - P
//   sum (z - P) = s0_t + n d,   sum (z - P)^2 = s1_t + 2 d s0_t + n d^2,
// the slabs are added in the order of k_bn_finish_v (1024 / CW groups, each every 1024 / CW-th slab, then bn_group_sums), and the
// batch mean, 1 / sqrt(var + eps) and the running pair follow as there.
template <int CW>
__global__ void __launch_bounds__(kBnFinishThreads)
k_bn_finish_slabs(const float* __restrict__ st, int nslab, int slab_rows, int C, int rows, float* __restrict__ mean,
                  float* __restrict__ rstd, float* __restrict__ run_mean, float* __restrict__ run_var, float mom) {
  constexpr int kBnFinishGroups = kBnFinishThreads / CW;
  __shared__ float sh[2][kBnFinishGroups][CW];
  const int lc = threadIdx.x % CW, q = threadIdx.x / CW;
  const int j = blockIdx.x * CW + lc;
  float a = 0.f, b = 0.f, P = 0.f;
  if (j < C) {
    const float* s0p = st + j;
    const float* s1p = st + (size_t)nslab * C + j;
    const float* pp = st + (size_t)2 * nslab * C + j;
    P = pp[0];
    const float n = (float)slab_rows;
    int s = q;
    for (; s + 3 * kBnFinishGroups < nslab; s += 4 * kBnFinishGroups) {      // twelve loads in flight
      float s0[4], s1[4], p[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const size_t o = (size_t)(s + u * kBnFinishGroups) * C;
        s0[u] = s0p[o]; s1[u] = s1p[o]; p[u] = pp[o];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const float d = p[u] - P;
        a += s0[u] + n * d;
        b += s1[u] + 2.f * d * s0[u] + n * d * d;
      }
    }
    for (; s < nslab; s += kBnFinishGroups) {
      const size_t o = (size_t)s * C;
      const float s0 = s0p[o], s1 = s1p[o], d = pp[o] - P;
      a += s0 + n * d;
      b += s1 + 2.f * d * s0 + n * d * d;
    }
  }
  sh[0][q][lc] = a; sh[1][q][lc] = b;
  __syncthreads();
  bn_group_sums<CW>(sh, q, lc, a, b);
  if (q != 0 || j >= C) return;
  const float inv = 1.f / (float)rows, m1 = a * inv;
  float var = b * inv - m1 * m1;
  var = var > 0.f ? var : 0.f;
  const float mu = P + m1;
  mean[j] = mu;
  rstd[j] = rsqrtf(var + kBnEpsV);
  if (run_mean) {   // running statistics take the unbiased batch variance
    const float unb = rows > 1 ? var * ((float)rows / (float)(rows - 1)) : var;
    run_mean[j] = (1.f - mom) * run_mean[j] + mom * mu;
    run_var[j] = (1.f - mom) * run_var[j] + mom * unb;
  }
}
// Few slabs: every block of the kernel that applies the statistics adds them up for itself, at the price of a read of all sums
// per block (at most 4096 per plane, from L2) and without the launch in between, which costs 4.4 us and a unit of a small
// network three of its fifteen launches.  Thread (channel j, group q): slabs q, q + G, ..., the groups' sums in order.
constexpr int kBnSmallC = 128, kBnSmallSums = 4096, kBnSmallBlocks = 512;
inline bool bn_small(int nslab, int C) { return C <= kBnSmallC && nslab * C <= kBnSmallSums; }
enum BnFinish { BN_GIVEN, BN_SHIFTED, BN_WIDE, BN_CONV };
struct BnSums {            // what the statistics come from, and where they go (block 0)
  const float* partial; int nslab, slab_rows, rows;
  float *mean, *rstd, *run_mean, *run_var; float mom;
};
template <typename A, class F>
__device__ __forceinline__ void bn_small_sums(int nslab, int C, A* sh, F add, A& a, A& b) {
  const int G = 256 / C, q = threadIdx.x / C, j = threadIdx.x - q * C;
  a = 0; b = 0;
  if (q < G) {
#pragma unroll 4
    for (int s = q; s < nslab; s += G) add(s, j, a, b);
    sh[q * C + j] = a;
    sh[256 + q * C + j] = b;
  }
  __syncthreads();
  if (q == 0) {
    a = 0; b = 0;
    for (int g = 0; g < G; ++g) { a += sh[g * C + j]; b += sh[256 + g * C + j]; }
  }
}
// Batch mean and 1 / sqrt(var + eps) of every channel into LDS; block 0 also leaves them in memory with the running pair.
template <BnFinish FIN>
__device__ __forceinline__ void bn_small_stats(const BnSums& t, const bf16_t* __restrict__ z, int C, float* mu_s, float* rs_s) {
  typedef typename std::conditional<FIN == BN_WIDE, double, float>::type A;
  __shared__ A sh[512];
  const size_t plane = (size_t)t.nslab * C;
  A a, b;
  float P = 0.f;
  if (FIN == BN_CONV && (int)threadIdx.x < 256 / C * C) P = t.partial[2 * plane + threadIdx.x % C];
  const float n = (float)t.slab_rows;
  bn_small_sums(t.nslab, C, sh, [&](int s, int j, A& x, A& y) {
    const float* p = t.partial + (size_t)s * C + j;
    if (FIN == BN_WIDE) {
      x += (A)p[0] + (A)p[2 * plane];
      y += (A)p[plane] + (A)p[3 * plane];
    } else if (FIN == BN_CONV) {
      const float d = p[2 * plane] - P, s0 = p[0];
      x += s0 + n * d;
      y += p[plane] + 2.f * d * s0 + n * d * d;
    } else {
      x += p[0];
      y += p[plane];
    }
  }, a, b);
  const int j = threadIdx.x;
  if (j < C) {
    float mu, var;
    if (FIN == BN_WIDE) {
      const A m1 = a / t.rows, v1 = b / t.rows - m1 * m1;
      mu = (float)m1;
      var = v1 < 0 ? 0.f : (float)v1;
    } else {
      const float inv = 1.f / (float)t.rows, m1 = (float)a * inv;
      var = (float)b * inv - m1 * m1;
      var = var > 0.f ? var : 0.f;
      mu = (FIN == BN_CONV ? P : (float)z[j]) + m1;
    }
    const float rs = rsqrtf(var + kBnEpsV);
    mu_s[j] = mu;
    rs_s[j] = rs;
    if (blockIdx.x == 0) {
      t.mean[j] = mu;
      t.rstd[j] = rs;
      if (t.run_mean) {   // running statistics take the unbiased batch variance
        const float unb = t.rows > 1 ? var * ((float)t.rows / (float)(t.rows - 1)) : var;
        t.run_mean[j] = (1.f - t.mom) * t.run_mean[j] + t.mom * mu;
        t.run_var[j] = (1.f - t.mom) * t.run_var[j] + t.mom * unb;
      }
    }
  }
  __syncthreads();
}
template <BnFinish FIN>
__global__ void __launch_bounds__(256) k_bn_apply_v(const bf16_t* __restrict__ z, const float* __restrict__ g,
                                                    const float* __restrict__ b, const bf16_t* __restrict__ res,
                                                    bf16_t* __restrict__ y, const float* __restrict__ mean,
                                                    const float* __restrict__ rstd, size_t nchunks, int C, int relu, BnSums t) {
  __shared__ __attribute__((aligned(16))) float mu_s[FIN ? kBnSmallC : 4], rs_s[FIN ? kBnSmallC : 4];
  if constexpr (FIN != BN_GIVEN) {
    bn_small_stats<FIN>(t, z, C, mu_s, rs_s);
    mean = mu_s; rstd = rs_s;
  }
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, st = (size_t)gridDim.x * 256;
  for (; i < nchunks; i += st) {
    const int c = (int)((i * 8) % C);
    float v[8], gg[8], bb[8], mu[8], rs[8];
    load8(z + i * 8, v); loadf8(g + c, gg); loadf8(b + c, bb); loadf8(mean + c, mu); loadf8(rstd + c, rs);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (v[e] - mu[e]) * rs[e] * gg[e] + bb[e];
    if (res) {
      float r[8];
      load8(res + i * 8, r);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += r[e];
    }
    if (relu) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
    }
    store8(y + i * 8, v);
  }
}
// SMALL: `sums` are the slabs' [2][nslab][C], added up here; block 0 leaves the shift and gain gradients in db and dg.
template <bool SMALL>
__global__ void __launch_bounds__(256) k_bn_bwd_apply_v(const bf16_t* __restrict__ dy, const bf16_t* __restrict__ yrelu,
                                                        const bf16_t* __restrict__ z, const float* __restrict__ mean,
                                                        const float* __restrict__ rstd, const float* __restrict__ g,
                                                        const float* __restrict__ sums, bf16_t* __restrict__ dz,
                                                        bf16_t* __restrict__ dres, size_t nchunks, int C, int rows,
                                                        int relu, int nslab, float* __restrict__ db, float* __restrict__ dg, int accumulate) {
  __shared__ __attribute__((aligned(16))) float tot[SMALL ? 2 * kBnSmallC : 4];
  __shared__ float sh[SMALL ? 512 : 4];
  if constexpr (SMALL) {
    const size_t plane = (size_t)nslab * C;
    float a, b;
    bn_small_sums(nslab, C, sh, [&](int s, int j, float& x, float& y) {
      x += sums[(size_t)s * C + j];
      y += sums[plane + (size_t)s * C + j];
    }, a, b);
    const int j = threadIdx.x;
    if (j < C) {
      tot[j] = a;
      tot[C + j] = b;
      if (blockIdx.x == 0 && db) {      // none: the caller wants the input gradient only
        db[j] = accumulate ? db[j] + a : a;
        dg[j] = accumulate ? dg[j] + b : b;
      }
    }
    __syncthreads();
    sums = tot;
  }
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x, st = (size_t)gridDim.x * 256;
  const float inv = 1.f / (float)rows;
  for (; i < nchunks; i += st) {
    const int c = (int)((i * 8) % C);
    float d[8], zz[8], mu[8], rs[8], gg[8], s0[8], s1[8], o[8];
    load8(dy + i * 8, d); load8(z + i * 8, zz);
    loadf8(mean + c, mu); loadf8(rstd + c, rs); loadf8(g + c, gg); loadf8(sums + c, s0); loadf8(sums + C + c, s1);
    if (relu) {
      float yy[8];
      load8(yrelu + i * 8, yy);
#pragma unroll
      for (int e = 0; e < 8; ++e) d[e] = yy[e] > 0.f ? d[e] : 0.f;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float xh = (zz[e] - mu[e]) * rs[e];
      o[e] = gg[e] * rs[e] * (d[e] - s0[e] * inv - xh * s1[e] * inv);
    }
    store8(dz + i * 8, o);
    if (dres) store8(dres + i * 8, d);
  }
}

// Rows per slab, given how many slabs the workspace holds.
int bn_slab(int rows, int C, size_t room) {
  int RL = 256 / (C / 8);
  int slab = (rows + 1023) / 1024;         // aim at about a thousand blocks
  int min_slab = RL * 4;                   // four rows in flight per thread
  if (slab < min_slab) slab = min_slab;
  if (room < (size_t)(rows + slab - 1) / slab) slab = (int)((rows + room - 1) / room);
  return slab;
}
// Slabs whose sums a caller's workspace has to hold, however the rows are cut here: slabs of eight rows per thread, or of the
// generic kernels' 1024 rows for the channel counts that are not bn_shifted.
size_t bn_least_slabs(int rows, int C) {
  int slab = 1024;
  if (bn_shifted(C)) {
    slab = (rows + 1023) / 1024;
    if (slab < 256 / (C / 8) * 8) slab = 256 / (C / 8) * 8;
  }
  return ((size_t)rows + slab - 1) / slab;
}
int blocks_for(size_t n) { size_t b = (n + 255) / 256; return (int)(b < 16384 ? b : 16384); }

}  // namespace

bool bn_fast_ok(const OpCtx& c, int rows, int C, const void* a, const void* b, const void* cc, const void* d) {
  if (c.dt != BF16 || C % 8 || C < 8 || C > 2048 || rows < 1) return false;
  return al16(a) && al16(b) && (!cc || al16(cc)) && (!d || al16(d));
}
// Does the workspace hold a slab's forward sums?  Where the generic kernels need less (one sum per slab at a time), they run.
bool bn_fwd_room(const OpCtx& c, int C) { return bn_shifted(C) || c.partial_elems >= (size_t)4 * C; }
hipError_t bn_fwd_fast(const OpCtx& c, const void* z, const float* g, const float* b, const void* res, void* y,
                       float* mean, float* rstd, int rows, int C, int relu, const BnRunning* run, const ConvStats* pre) {
  const bool given = run && run->use;   // mean / rstd already hold the statistics to normalise with
  float* rm = run ? run->mean : nullptr;
  float* rv = run ? run->var : nullptr;
  const float mom = run ? run->momentum : 0.f;
  const size_t nch = (size_t)rows * C / 8;
  BnSums t = {c.partial, 0, 0, rows, mean, rstd, rm, rv, mom};
  auto apply = [&](auto fin) {
    constexpr BnFinish FIN = decltype(fin)::value;
    int blocks = blocks_for(nch);
    if (FIN != BN_GIVEN && blocks > kBnSmallBlocks) blocks = kBnSmallBlocks;
    k_bn_apply_v<FIN><<<blocks, 256, 0, c.stream>>>((const bf16_t*)z, g, b, (const bf16_t*)res, (bf16_t*)y, mean, rstd, nch, C, relu, t);
    return hipGetLastError();
  };
  typedef std::integral_constant<BnFinish, BN_SHIFTED> Shifted;
  typedef std::integral_constant<BnFinish, BN_WIDE> Wide;
  typedef std::integral_constant<BnFinish, BN_CONV> Conv;
  if (!given && pre && pre->nslab > 0 && (size_t)pre->nslab * pre->slab_rows == (size_t)rows) {
    // the convolution in front left the per-slab sums: no pass over z for the statistics
    t.partial = pre->buf; t.nslab = pre->nslab; t.slab_rows = pre->slab_rows;
    if (bn_small(t.nslab, C)) return apply(Conv{});
    if (pre->nslab >= kBnManySlabs)
      k_bn_finish_slabs<16><<<(C + 15) / 16, kBnFinishThreads, 0, c.stream>>>(pre->buf, pre->nslab, pre->slab_rows, C, rows, mean, rstd, rm, rv, mom);
    else
      k_bn_finish_slabs<64><<<(C + 63) / 64, kBnFinishThreads, 0, c.stream>>>(pre->buf, pre->nslab, pre->slab_rows, C, rows, mean, rstd, rm, rv, mom);
  } else if (!given && !bn_shifted(C)) {
    if (bn_least_slabs(rows, C) * C > c.partial_elems) return hipErrorInvalidValue;
    // at most a slab per compute unit: two blocks add up all of 65536 x 96's sums, 13.7 us with 512 slabs, 7.3 us with 256
    const size_t room = c.partial_elems / ((size_t)4 * C);
    const int slab = bn_slab(rows, C, room < 256 ? room : 256), nslab = (rows + slab - 1) / slab;
    const size_t shm = (size_t)2 * (256 / (C / 8)) * C * sizeof(double);
    k_bn_partial_v<2><<<nslab, 256, shm, c.stream>>>((const bf16_t*)z, nullptr, nullptr, nullptr, nullptr, c.partial, rows, C,
                                                     slab, 0);
    t.nslab = nslab;
    if (bn_small(nslab, C)) return apply(Wide{});
    if (nslab >= kBnManySlabs)
      k_bn_finish_wide<16><<<(C + 15) / 16, kBnFinishThreads, 0, c.stream>>>(c.partial, nslab, C, rows, mean, rstd, rm, rv, mom);
    else
      k_bn_finish_wide<64><<<(C + 63) / 64, kBnFinishThreads, 0, c.stream>>>(c.partial, nslab, C, rows, mean, rstd, rm, rv, mom);
  } else if (!given) {
    if (2 * bn_least_slabs(rows, C) * C > c.partial_elems) return hipErrorInvalidValue;
    const int slab = bn_slab(rows, C, c.partial_elems / ((size_t)2 * C)), nslab = (rows + slab - 1) / slab;
    const int RL = 256 / (C / 8);
    const size_t shm = (size_t)2 * RL * C * sizeof(float);
    k_bn_partial_v<0><<<nslab, 256, shm, c.stream>>>((const bf16_t*)z, nullptr, (const bf16_t*)z, nullptr, nullptr,
                                                     c.partial, rows, C, slab, 0);
    t.nslab = nslab;
    // not in place: the blocks take their pivots from row 0 of z, which block 0 has written by then
    if (bn_small(nslab, C) && y != z) return apply(Shifted{});
    if (nslab >= kBnManySlabs)
      k_bn_finish_v<16><<<(C + 15) / 16, kBnFinishThreads, 0, c.stream>>>(c.partial, nslab, C, rows, (const bf16_t*)z, mean, rstd, 0, rm, rv, mom);
    else
      k_bn_finish_v<64><<<(C + 63) / 64, kBnFinishThreads, 0, c.stream>>>(c.partial, nslab, C, rows, (const bf16_t*)z, mean, rstd, 0, rm, rv, mom);
  }
  return apply(std::integral_constant<BnFinish, BN_GIVEN>{});
}
hipError_t bn_bwd_fast(const OpCtx& c, const void* dy, const void* y, const void* z, const float* mean,
                       const float* rstd, const float* g, void* dz, void* dres, float* dg, float* db, int rows, int C,
                       int relu, int accumulate) {
  if ((2 * bn_least_slabs(rows, C) + 2) * C > c.partial_elems) return hipErrorInvalidValue;
  const int slab = bn_slab(rows, C, c.partial_elems / ((size_t)2 * C) - 1), nslab = (rows + slab - 1) / slab;
  float* sums = c.partial + (size_t)2 * nslab * C;
  const int RL = 256 / (C / 8);
  const size_t shm = (size_t)2 * RL * C * sizeof(float);
  k_bn_partial_v<1><<<nslab, 256, shm, c.stream>>>((const bf16_t*)dy, (const bf16_t*)y, (const bf16_t*)z, mean, rstd,
                                                   c.partial, rows, C, slab, relu);
  const size_t nch = (size_t)rows * C / 8;
  if (bn_small(nslab, C)) {
    const int blocks = blocks_for(nch) < kBnSmallBlocks ? blocks_for(nch) : kBnSmallBlocks;
    k_bn_bwd_apply_v<true><<<blocks, 256, 0, c.stream>>>((const bf16_t*)dy, (const bf16_t*)y, (const bf16_t*)z, mean, rstd, g, c.partial,
                                                         (bf16_t*)dz, (bf16_t*)dres, nch, C, rows, relu, nslab, db, dg, accumulate);
    return hipGetLastError();
  }
  if (nslab >= kBnManySlabs)
    k_bn_finish_v<16><<<(C + 15) / 16, kBnFinishThreads, 0, c.stream>>>(c.partial, nslab, C, rows, nullptr, sums, sums + C, 1, db, dg, accumulate ? 1.f : 0.f);
  else
    k_bn_finish_v<64><<<(C + 63) / 64, kBnFinishThreads, 0, c.stream>>>(c.partial, nslab, C, rows, nullptr, sums, sums + C, 1, db, dg, accumulate ? 1.f : 0.f);
  k_bn_bwd_apply_v<false><<<blocks_for(nch), 256, 0, c.stream>>>((const bf16_t*)dy, (const bf16_t*)y, (const bf16_t*)z, mean, rstd, g, sums,
                                                                (bf16_t*)dz, (bf16_t*)dres, nch, C, rows, relu, 0, nullptr, nullptr, 0);
  return hipGetLastError();
}

}  // namespace lp
