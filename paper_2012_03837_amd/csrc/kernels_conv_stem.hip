// The stem: a 3x3 convolution (stride 1, padding 1) of an image with one to three channels, bf16, forward and filter
// gradient, on the matrix cores.  As an implicit GEMM over gathered operands its reduction (9 C <= 27 taps) is shorter
// than the gather's index arithmetic; here a block keeps a band of image rows with its zero border in LDS and every
// fragment element is one 2-byte LDS read at a per-lane constant offset, so both kernels are bound by the one large
// tensor they write or read (z or dz: 2 bytes per output element).
// 256 x 32 x 32 x 3 -> 64 channels (33.6 MB): forward 35 -> 17 us and no statistics pass behind it (7 us), filter gradient 418 + 23 -> 13 + 5 us.
#include "common.h"
#include "gemm_common.h"

namespace lp {

hipError_t op_reduce_partials(const OpCtx& c, const float* partial, int nblk, int n, float* out, int accumulate);

namespace {

typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

struct StemShape {
  int H, W, C, O;      // image, channels in and out
  int RB, chunks;      // image rows per block, blocks per image
  int LW;              // pixels per LDS row
};

// Output column of row i of the n-side fragment, so that a lane's accumulators are runs of 8 consecutive columns
// (as in the other MFMA kernels).
__device__ __forceinline__ int nmap(int i) {
  const int g = i >> 3, h = (i >> 2) & 1, j = i & 3;
  return 16 * (g >> 1) + 8 * h + 4 * (g & 1) + j;
}

// Image rows h0 - 1 .. h0 + rb of one image, pixels -1 .. LW - 2 of each, zero outside the image.
__device__ __forceinline__ void load_band(bf16_t* xs, const bf16_t* __restrict__ x, const StemShape& s, int n, int h0, int rb) {
  const int per_row = s.LW * s.C, total = (rb + 2) * per_row;
  for (int i = threadIdx.x; i < total; i += 256) {
    const int r = i / per_row, t = i - r * per_row;
    const int h = h0 + r - 1, e = t - s.C;            // element of the image row
    const bool ok = h >= 0 && h < s.H && e >= 0 && e < s.W * s.C;
    xs[i] = ok ? x[((size_t)n * s.H + h) * s.W * s.C + e] : (bf16_t)0.f;
  }
}

// Forward.  Block: a band of RB image rows; a wave takes every fourth run of 32 output pixels and 64 output channels
// at a time (blockIdx.y).  Weights sit in registers (k past the taps is zero), a pixel's 27 taps are read from the
// band (its slots past the taps are cleared too: an infinite pixel against a zero weight would be a NaN), results leave
// through a 4 KB patch as whole lines.  STATS (bands of equal size, whole runs, the same number
// per wave): the column sums the normalisation needs, per band (see ConvStats).
template <bool STATS>
__global__ void __launch_bounds__(256) k_stem_fwd(const bf16_t* __restrict__ x, const bf16_t* __restrict__ w,
                                                  bf16_t* __restrict__ out, StemShape s, float* __restrict__ stats,
                                                  int nslab) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  char* patch = sm + (threadIdx.x >> 6) * 4096;
  bf16_t* xs = reinterpret_cast<bf16_t*>(sm + 4 * 4096);
  const int n = blockIdx.x / s.chunks, h0 = (blockIdx.x % s.chunks) * s.RB;
  const int rb = h0 + s.RB < s.H ? s.RB : s.H - h0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, hf = lane >> 5, K = 9 * s.C, n0 = blockIdx.y * 64;
  bf16x8 fw[2][2];
  int off[2][8];
  u16x8 live[2];             // all ones for the slots that hold a tap
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = 16 * ks + 8 * hf + e, kk = k < K ? k : 0;
      live[ks][e] = k < K ? 0xffff : 0;
      const int r = kk / (3 * s.C);
      off[ks][e] = r * s.LW * s.C + (kk - r * 3 * s.C);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int col = n0 + 32 * i + nmap(li);
        fw[i][ks][e] = (k < K && col < s.O) ? w[(size_t)col * K + k] : (bf16_t)0.f;
      }
    }
  load_band(xs, x, s, n, h0, rb);
  __syncthreads();
  const int px = rb * s.W, runs = (px + 31) / 32;
  const int rr = lane >> 3, rc = lane & 7;
  float s0 = 0.f, s1 = 0.f, piv = 0.f;
  bf16_t* ob = out + ((size_t)n * s.H + h0) * s.W * s.O + n0 + 8 * rc;
  for (int t = wave; t < runs; t += 4) {
    const int pi = 32 * t + li < px ? 32 * t + li : px - 1;
    const int p = pi / s.W, q = pi - p * s.W;
    const bf16_t* base = xs + (p * s.LW + q) * s.C;
    f32x16 acc[2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      bf16x8 fx;
#pragma unroll
      for (int e = 0; e < 8; ++e) fx[e] = base[off[ks][e]];
      fx = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u16x8, fx) & live[ks]);
#pragma unroll
      for (int i = 0; i < 2; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[i][ks], fx, acc[i], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (bf16_t)acc[i][8 * h + e];
        *reinterpret_cast<bf16x8*>(patch + li * 128 + (((4 * i + 2 * h + hf) ^ ((li >> 1) & 7)) << 4)) = v;
      }
#pragma unroll
    for (int I = 0; I < 4; ++I) {
      const int r = 8 * I + rr, pix = 32 * t + r;
      if (pix < px && n0 + 8 * rc < s.O)
        *reinterpret_cast<bf16x8*>(ob + (size_t)pix * s.O) =
            *reinterpret_cast<const bf16x8*>(patch + r * 128 + ((rc ^ ((r >> 1) & 7)) << 4));
    }
    if (STATS) {
#pragma unroll
      for (int r = 0; r < 32; ++r) {
        const float v = (float)*reinterpret_cast<const bf16_t*>(patch + r * 128 + (((lane >> 3) ^ ((r >> 1) & 7)) << 4) + (lane & 7) * 2);
        if (r == 0 && t == wave) piv = v;
        const float d = v - piv;
        s0 += d; s1 += d * d;
      }
    }
  }
  if (STATS) {         // the waves' sums, shifted to the first wave's pivot and added in wave order
    float* mine = reinterpret_cast<float*>(patch);
    mine[lane] = s0; mine[64 + lane] = s1; mine[128 + lane] = piv;
    __syncthreads();
    if (wave == 0 && n0 + lane < s.O) {
      const float cnt = (float)(px / 4);
#pragma unroll
      for (int u = 1; u < 4; ++u) {
        const float* o = reinterpret_cast<const float*>(sm + u * 4096);
        const float o0 = o[lane], o1 = o[64 + lane], d = o[128 + lane] - piv;
        s0 += o0 + cnt * d;
        s1 += o1 + 2.f * d * o0 + cnt * d * d;
      }
      float* sp = stats + (size_t)blockIdx.x * s.O + n0 + lane;
      sp[0] = s0;
      sp[(size_t)nslab * s.O] = s1;
      sp[(size_t)2 * nslab * s.O] = piv;
    }
  }
}

// Filter gradient: dw[o, j] = sum over pixels of dz[pixel, o] * x[pixel + tap j].  Block: a band of image rows and 64
// output channels; the reduction index is the pixel, 16 at a time along an image row (a row is rounded up to 16, a run to
// four steps: both operands are zero there, because a real pixel's infinity against a zero of dz would be a NaN).  A wave takes every fourth run of 64 pixels: dz goes through a wave-private 8 KB LDS tile and is read
// transposed (ds_read_b64_tr_b16), the next run's loads in flight meanwhile; the taps of 8 consecutive pixels are
// eight 2-byte reads of the band.  The four waves' sums are added in order, the blocks' by k_reduce_partials.
__global__ void __launch_bounds__(256) k_stem_wgrad(const bf16_t* __restrict__ dz, const bf16_t* __restrict__ x,
                                                    float* __restrict__ ws, StemShape s) {
  extern __shared__ __attribute__((aligned(16))) char sm[];
  bf16_t* xs = reinterpret_cast<bf16_t*>(sm + 4 * 8192);
  const int n = blockIdx.x / s.chunks, h0 = (blockIdx.x % s.chunks) * s.RB;
  const int rb = h0 + s.RB < s.H ? s.RB : s.H - h0;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 31, hf = lane >> 5, J = 9 * s.C, n0 = blockIdx.y * 64;
  bf16_t* tile = reinterpret_cast<bf16_t*>(sm + wave * 8192);      // [64 pixels][64 channels]
  load_band(xs, x, s, n, h0, rb);
  __syncthreads();
  const int steps_row = (s.W + 15) / 16, steps = rb * steps_row;   // 16-pixel steps of the band
  const int jj = li < J ? li : 0, jr = jj / (3 * s.C), joff = jr * s.LW * s.C + (jj - jr * 3 * s.C);
  const int ch = lane & 7, pr = lane >> 3;
  const bool col_ok = n0 + 8 * ch < s.O;
  const bf16_t* zb = dz + ((size_t)n * s.H + h0) * s.W * s.O + n0 + 8 * (col_ok ? ch : 0);
  f32x16 acc[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
  bf16x8 zr[8];
  auto fetch = [&](int t0) {            // pixels of steps t0 .. t0 + 3: instruction i carries rows 8 i + lane / 8
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int st = t0 + (i >> 1), p = st / steps_row, q = (st - p * steps_row) * 16 + (i & 1) * 8 + pr;
      const bool ok = st < steps && q < s.W && col_ok;
      zr[i] = *reinterpret_cast<const bf16x8*>(zb + (ok ? (size_t)(p * s.W + q) * s.O : 0));
      if (!ok) {
#pragma unroll
        for (int e = 0; e < 8; ++e) zr[i][e] = (bf16_t)0.f;
      }
    }
  };
  if (4 * wave < steps) fetch(4 * wave);
  // fragment rows of the transposing read: 16-lane group's 16-row half, chunk of 4 rows
  const int rowb = 16 * ((lane >> 4) & 1) + 4 * (lane & 3), kb = 8 * hf + ((lane & 15) >> 2);
  for (int t0 = 4 * wave; t0 < steps; t0 += 16) {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<bf16x8*>(tile + (8 * i + pr) * 64 + 8 * (ch ^ ((pr & 3) << 1))) = zr[i];
    if (t0 + 16 < steps) fetch(t0 + 16);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int st = t0 + u < steps ? t0 + u : steps - 1, p = st / steps_row, q = (st - p * steps_row) * 16 + 8 * hf;
      const bf16_t* xb = xs + (p * s.LW + q) * s.C + joff;
      bf16x8 fx;
#pragma unroll
      for (int e = 0; e < 8; ++e) fx[e] = xb[e * s.C];
      const int left = t0 + u < steps ? s.W - (q - 8 * hf) : 0;      // pixels of the step inside the row (wave-uniform)
      if (left < 16) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (8 * hf + e >= left) fx[e] = (bf16_t)0.f;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        // chunk c of pixel row k sits in slot c ^ ((k & 3) << 1): the four rows of a read fall on different banks
        const int k = 16 * u + kb, row = 32 * i + rowb;
        const bf16_t* p0 = tile + k * 64 + 8 * ((row >> 3) ^ ((k & 3) << 1)) + (row & 7);
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p0);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p0 + 4 * 64));
        bf16x8 fz;
#pragma unroll
        for (int e = 0; e < 4; ++e) { fz[e] = lo[e]; fz[4 + e] = hi[e]; }
        acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fz, fx, acc[i], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // the tile has been read before it is filled again
  }
  __syncthreads();
  // accumulator v of lane (li, hf): output channel 32 i + 8 (v / 4) + 4 hf + v % 4, tap li
  float* red = reinterpret_cast<float*>(sm);                 // [4 waves][64 channels][32 taps]
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) red[(wave * 64 + 32 * i + 8 * (v >> 2) + 4 * hf + (v & 3)) * 32 + li] = acc[i][v];
  __syncthreads();
  for (int i = threadIdx.x; i < 64 * 32; i += 256) {
    const int o = i >> 5, j = i & 31;
    if (j < J && n0 + o < s.O)
      ws[((size_t)blockIdx.x * s.O + n0 + o) * J + j] = ((red[i] + red[2048 + i]) + red[4096 + i]) + red[6144 + i];
  }
}

// Image rows per block: about 512 blocks, bands of at least 128 pixels that fit 24 KB of LDS, and a divisor of H where
// one lies between half of that and that (bands of one size can carry the normalisation's statistics).
StemShape stem_shape(const ConvArgs& a, int lds_width) {
  StemShape s;
  s.H = a.H; s.W = a.W; s.C = a.C; s.O = a.O; s.LW = lds_width;
  int rb = (int)((size_t)a.N * a.H / 512);
  const int least = (127 + a.W) / a.W, most = 24 * 1024 / (lds_width * a.C * 2) - 2;
  if (rb < least) rb = least;
  if (rb > most) rb = most;
  if (rb > a.H) rb = a.H;
  if (rb < 1) rb = 1;
  for (int d = rb; 2 * d >= rb && d >= 1; --d)
    if (a.H % d == 0) { rb = d; break; }
  s.RB = rb; s.chunks = (a.H + rb - 1) / rb;
  return s;
}
size_t band_bytes(const StemShape& s) { return (((size_t)(s.RB + 2) * s.LW * s.C * 2) + 15) & ~(size_t)15; }

}  // namespace

bool conv_stem_ok(const OpCtx& c, const ConvArgs& a, const void* p0, const void* p1) {
  return c.dt == BF16 && a.C >= 1 && a.C <= 3 && a.R == 3 && a.S == 3 && a.stride == 1 && a.pad == 1 && a.O % 8 == 0 &&
         a.N >= 1 && (a.W + 18) * a.C * 2 * 3 <= 24 * 1024 && (size_t)a.N * a.H < ((size_t)1 << 31) && ((uintptr_t)p0 & 15) == 0 && ((uintptr_t)p1 & 15) == 0;
}

hipError_t conv_stem_fwd(const OpCtx& c, const ConvArgs& a, const void* x, const void* w, void* out, ConvStats* st) {
  const StemShape s = stem_shape(a, a.W + 2);
  const dim3 grid(a.N * s.chunks, (a.O + 63) / 64);
  const size_t shm = 4 * 4096 + band_bytes(s);
  const int nslab = a.N * s.chunks;
  if (st && st->buf && a.H % s.RB == 0 && s.RB * a.W % 128 == 0 && (size_t)3 * nslab * a.O <= st->cap) {
    st->nslab = nslab; st->slab_rows = s.RB * a.W;
    k_stem_fwd<true><<<grid, 256, shm, c.stream>>>((const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, s, st->buf, nslab);
  } else {
    k_stem_fwd<false><<<grid, 256, shm, c.stream>>>((const bf16_t*)x, (const bf16_t*)w, (bf16_t*)out, s, nullptr, 0);
  }
  return hipGetLastError();
}

// Returns hipErrorInvalidValue, with nothing launched, if the workspace cannot hold a table of every block's sums.
hipError_t conv_stem_wgrad(const OpCtx& c, const ConvArgs& a, const void* dout, const void* x, float* dw, int accumulate) {
  const StemShape s = stem_shape(a, (a.W + 15) / 16 * 16 + 2);
  const int blocks = a.N * s.chunks, J = 9 * a.C;
  if (!c.splitk_ws || (size_t)blocks * a.O * J > c.splitk_elems) return hipErrorInvalidValue;
  k_stem_wgrad<<<dim3(blocks, (a.O + 63) / 64), 256, 4 * 8192 + band_bytes(s), c.stream>>>((const bf16_t*)dout, (const bf16_t*)x,
                                                                                       c.splitk_ws, s);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return op_reduce_partials(c, c.splitk_ws, blocks, a.O * J, dw, accumulate);
}

}  // namespace lp
