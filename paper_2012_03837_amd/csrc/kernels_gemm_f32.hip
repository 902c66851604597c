// Products in fp32 arithmetic (v_mfma_f32_16x16x4_f32: exact fp32 products and sums) for fp32 and for every bf16 shape
// the bf16 matrix kernels do not take (unaligned rows, a 10-class head).  The problems are small: a block's four waves
// each take a quarter of the reduction of one (16 T) x (16 T) tile, fragments go from global memory straight to
// registers, several 16-deep chunks in flight, and the four partial tiles are added in wave order through LDS.  No
// operand staging and no barrier in the loop, so a product is one or two memory latencies, its matrix instructions and
// the reduction.
//
// A chunk is 16 k: lane (i = lane % 16, g = lane / 16) holds k = 4 g .. 4 g + 3 of row i, and the j-th of the chunk's
// four matrix instructions takes element j of every lane.  Both operands use this order, so any storage layout pairs
// with any other: k contiguous is one 16-byte (bf16: 8-byte) load per row and chunk, k-major four 4-byte loads.
//
// Up to four independent products share a launch (GemmArgs::rowsum adds a bias gradient to a weight gradient: sums of
// A's rows, taken from the fragments by the blocks of the first tile column).
//   128 x 256 x 256 fp32 (a layer of the MLP): 12.1 -> 4.5 us; 333 x 1000 x 520: 42 -> 12 us;
//   1024 x 1024 x 1024: 160 -> 33 us (the 64 x 64 x 32 FMA kernel before).
#include <stdio.h>
#include "common.h"
#include "gemm_common.h"

namespace lp {

namespace {

constexpr int kMaxFGroup = 4;

template <typename T>
struct FProblem {
  const T* A; const T* B;
  int64_t lda, ldb;
  int a_kc, b_kc, a_vec, b_vec;      // vec: rows start on whole 4-element loads
  int M, N, K;
  int first, tiles_n;                // first tile number of this problem, tile columns
  float* rowsum;
  Epilogue e;
};
template <typename T, int NP>
struct FGroup { FProblem<T> p[NP]; int n; };

typedef float f4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f4 load4(const float* p) { return *reinterpret_cast<const f4*>(p); }
__device__ __forceinline__ f4 load4(const bf16_t* p) {
  const bf16x4 v = *reinterpret_cast<const bf16x4*>(p);
  f4 r = {(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
  return r;
}

// One lane's four elements of a 16-deep chunk.  `base` points at (row, k = 0) of this lane's row; MASK: some k of the
// chunk may lie past k_hi (clamped for the load, zeroed after it).
template <bool MASK, typename T>
__device__ __forceinline__ f4 fetch4(const T* base, int64_t ld, int kc, int vec, int k, int k_hi) {
  f4 r;
  if (kc && vec && (!MASK || k + 4 <= k_hi)) {
    r = load4(base + k);
  } else {
    const int64_t st = kc ? 1 : ld;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kk = MASK ? (k + j < k_hi ? k + j : k_hi - 1) : k + j;
      r[j] = to_f(base[kk * st]);
    }
    if (MASK) {
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = k + j < k_hi ? r[j] : 0.f;
    }
  }
  return r;
}

template <typename T, int TT, int NP>
__global__ void __launch_bounds__(256) k_gemm_f(FGroup<T, NP> grp) {
  constexpr int EDGE = 16 * TT, LDP = EDGE + 4;       // LDS rows of a partial tile
  constexpr int DEPTH = TT == 4 ? 1 : (TT == 2 ? 2 : 4);       // chunks per register set
  extern __shared__ __attribute__((aligned(16))) float part[];      // [4][EDGE][LDP], then [4][EDGE] row sums
  int pi = 0;
#pragma unroll
  for (int i = 1; i < NP; ++i)
    if (i < grp.n && (int)blockIdx.x >= grp.p[i].first) pi = i;
  const FProblem<T>& P = grp.p[pi];
  const int tile = blockIdx.x - P.first, tm = tile / P.tiles_n, tn = tile - tm * P.tiles_n;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int K = P.K, kq = ((K + 3) / 4 + 15) & ~15;     // a wave's share of the reduction: whole chunks
  const int k_lo = wave * kq, k_hi = k_lo + kq < K ? k_lo + kq : K;
  const T *ap[TT], *bp[TT];
#pragma unroll
  for (int t = 0; t < TT; ++t) {
    int m = tm * EDGE + 16 * t + li, n = tn * EDGE + 16 * t + li;
    m = m < P.M ? m : P.M - 1;
    n = n < P.N ? n : P.N - 1;
    ap[t] = P.A + (P.a_kc ? (int64_t)m * P.lda : (int64_t)m);
    bp[t] = P.B + (P.b_kc ? (int64_t)n * P.ldb : (int64_t)n);
  }
  const bool sums = P.rowsum && tn == 0;
  f4 acc[TT][TT];
  float rs[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) {
    rs[i] = 0.f;
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  }
  f4 a0[DEPTH][TT], b0[DEPTH][TT], a1[DEPTH][TT], b1[DEPTH][TT];
  auto fetch = [&](f4 (&a)[DEPTH][TT], f4 (&b)[DEPTH][TT], int k0) {
    if (k0 + 16 * DEPTH <= k_hi) {
#pragma unroll
      for (int c = 0; c < DEPTH; ++c)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          a[c][t] = fetch4<false>(ap[t], P.lda, P.a_kc, P.a_vec, k0 + 16 * c + 4 * g, k_hi);
          b[c][t] = fetch4<false>(bp[t], P.ldb, P.b_kc, P.b_vec, k0 + 16 * c + 4 * g, k_hi);
        }
    } else {
#pragma unroll
      for (int c = 0; c < DEPTH; ++c)
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          a[c][t] = fetch4<true>(ap[t], P.lda, P.a_kc, P.a_vec, k0 + 16 * c + 4 * g, k_hi);
          b[c][t] = fetch4<true>(bp[t], P.ldb, P.b_kc, P.b_vec, k0 + 16 * c + 4 * g, k_hi);
        }
    }
  };
  auto mma = [&](const f4 (&a)[DEPTH][TT], const f4 (&b)[DEPTH][TT]) {
#pragma unroll
    for (int c = 0; c < DEPTH; ++c) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int x = 0; x < TT; ++x)
#pragma unroll
          for (int y = 0; y < TT; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][x][j], b[c][y][j], acc[x][y], 0, 0, 0);
      if (sums) {
#pragma unroll
        for (int x = 0; x < TT; ++x) rs[x] += (a[c][x][0] + a[c][x][1]) + (a[c][x][2] + a[c][x][3]);
      }
    }
  };
  if (k_lo < k_hi) {
    constexpr int STEP = 16 * DEPTH;
    fetch(a0, b0, k_lo);
    int k0 = k_lo;
    for (; k0 + STEP < k_hi; k0 += 2 * STEP) {       // two register sets, loads one set ahead
      fetch(a1, b1, k0 + STEP);
      mma(a0, b0);
      if (k0 + 2 * STEP < k_hi) fetch(a0, b0, k0 + 2 * STEP);
      mma(a1, b1);
    }
    if (k0 < k_hi) mma(a0, b0);
  }
  // partial tiles: accumulator v of lane (li, g) is row 4 g + v, column li of its 16 x 16 tile
  float* mine = part + (size_t)wave * EDGE * LDP;
#pragma unroll
  for (int x = 0; x < TT; ++x)
#pragma unroll
    for (int y = 0; y < TT; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) mine[(16 * x + 4 * g + v) * LDP + 16 * y + li] = acc[x][y][v];
  float* rsum = part + (size_t)4 * EDGE * LDP;
  if (sums) {
#pragma unroll
    for (int x = 0; x < TT; ++x) {
      rs[x] += __shfl_xor(rs[x], 16, 64);
      rs[x] += __shfl_xor(rs[x], 32, 64);
      if (g == 0) rsum[wave * EDGE + 16 * x + li] = rs[x];
    }
  }
  __syncthreads();
  constexpr int PT = EDGE * LDP;
#pragma unroll 1
  for (int i = threadIdx.x; i < EDGE * EDGE; i += 256) {
    const int r = i / EDGE, col = i % EDGE, m = tm * EDGE + r, n = tn * EDGE + col;
    if (m < P.M && n < P.N) {
      const float* q = part + r * LDP + col;
      epilogue_store<T>(P.e, m, n, (q[0] + q[PT]) + (q[2 * PT] + q[3 * PT]));
    }
  }
  if (sums && (int)threadIdx.x < EDGE) {
    const int m = tm * EDGE + threadIdx.x;
    if (m < P.M) {
      const float* q = rsum + threadIdx.x;
      const float v = (q[0] + q[EDGE]) + (q[2 * EDGE] + q[3 * EDGE]);
      P.rowsum[m] = P.e.accumulate ? P.rowsum[m] + v : v;
    }
  }
}

template <typename T, int TT, int NP>
hipError_t launch_f(const OpCtx& c, FGroup<T, NP>& grp) {
  int tiles = 0;
  for (int i = 0; i < grp.n; ++i) {
    FProblem<T>& p = grp.p[i];
    p.first = tiles;
    p.tiles_n = (p.N + 16 * TT - 1) / (16 * TT);
    tiles += p.tiles_n * ((p.M + 16 * TT - 1) / (16 * TT));
  }
  constexpr int EDGE = 16 * TT;
  constexpr size_t shm = (size_t)(4 * EDGE * (EDGE + 4) + 4 * EDGE) * sizeof(float);
  static bool configured = false;
  if (shm > 64 * 1024 && !configured) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(k_gemm_f<T, TT, NP>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return e;
    configured = true;
  }
  k_gemm_f<T, TT, NP><<<tiles, 256, shm, c.stream>>>(grp);
  return hipGetLastError();
}

// Tile edge: the largest of 64, 32, 16 that still gives the chip's 256 compute units a tile each (32: half of them; a
// tile's traffic grows with 1 / edge, its time with the square).  Measured on 333 x 1000 x 520 (84 / 352 / 1323 tiles):
// 22 / 12 / 15 us; 128 x 256 x 256 (8 / 32 / 128 tiles): 11 / 6.5 / 4.5 us.
template <typename T, int NP>
hipError_t gemm_f_t(const OpCtx& c, const GemmArgs* gs, int n) {
  FGroup<T, NP> grp = {};
  long t64 = 0, t32 = 0;
  constexpr int al = 4 * (int)sizeof(T) - 1;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = gs[i];
    const int N = g.b_rows && g.b_rows < g.N ? g.b_rows : g.N;      // element by element: no padding columns
    if (g.M <= 0 || N <= 0) continue;
    FProblem<T>& p = grp.p[grp.n++];
    p.A = (const T*)g.A; p.B = (const T*)g.B; p.lda = g.lda; p.ldb = g.ldb;
    p.a_kc = g.a_kc; p.b_kc = g.b_kc;
    p.a_vec = g.lda % 4 == 0 && ((uintptr_t)g.A & al) == 0;
    p.b_vec = g.ldb % 4 == 0 && ((uintptr_t)g.B & al) == 0;
    p.M = g.M; p.N = N; p.K = g.K; p.rowsum = g.rowsum;
    p.e = make_epilogue(g);
    t64 += (long)((g.M + 63) / 64) * ((N + 63) / 64);
    t32 += (long)((g.M + 31) / 32) * ((N + 31) / 32);
  }
  if (grp.n == 0) return hipSuccess;
  if (t64 >= 256) return launch_f<T, 4, NP>(c, grp);
  if (t32 >= 128) return launch_f<T, 2, NP>(c, grp);
  return launch_f<T, 1, NP>(c, grp);
}

}  // namespace

hipError_t gemm_f32(const OpCtx& c, const GemmArgs* gs, int n) {
  if (n == 1) return c.dt == BF16 ? gemm_f_t<bf16_t, 1>(c, gs, 1) : gemm_f_t<float, 1>(c, gs, 1);
  for (int i = 0; i < n; i += kMaxFGroup) {
    const int k = n - i < kMaxFGroup ? n - i : kMaxFGroup;
    hipError_t e = c.dt == BF16 ? gemm_f_t<bf16_t, kMaxFGroup>(c, gs + i, k) : gemm_f_t<float, kMaxFGroup>(c, gs + i, k);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lp
