// Products in fp32 arithmetic (v_mfma_f32_16x16x4_f32: exact fp32 products and sums) for fp32 and for every bf16 shape
// the bf16 matrix kernels do not take (unaligned rows, a 10-class head).  The problems are small: a block's four waves
// each take a quarter of the reduction of one (16 T) x (16 T) tile, fragments go from global memory straight to
// registers, several 16-deep chunks in flight, and the four partial tiles are added in wave order through LDS.  No
// operand staging and no barrier in the loop, so a product is one or two memory latencies, its matrix instructions and
// the reduction.
//
// A chunk is 16 k: lane (i = lane % 16, g = lane / 16) holds k = 4 g .. 4 g + 3 of row i, and the j-th of the chunk's
// four matrix instructions takes element j of every lane.  Both operands use this order, so any storage layout pairs
// with any other: k contiguous is one 16-byte (bf16: 8-byte) load per row and chunk; k-major is one load of the T neighbouring
// rows that a lane then owns, T i .. T i + T - 1 instead of i, 16 + i, ... (rows in whole T-element loads), or four
// one-element loads per row.  The former only in 64-wide tiles, where a weight gradient otherwise issues 32 loads of 4 bytes per
// chunk, each with 64-bit address arithmetic (a step of six layers of 520 and 1000 with a batch of 333: 478 -> 443 us);
// in the smaller ones, which are latencies and not loads, more forms of the code cost what they save (61.5 -> 63.8 us,
// four layers of 256).
//
// Up to sixteen independent products share a launch (GemmArgs::rowsum adds a bias gradient to a weight gradient: sums of
// A's rows, taken from the fragments by the blocks of the first tile column).
//   128 x 256 x 256 fp32 (a layer of the MLP): 12.1 -> 4.2 us; 333 x 1000 x 520: 42 -> 11.6 us;
//   1024 x 1024 x 1024: 29 us (74 TFLOP/s), 4096 cubed 1.64 ms (84 TFLOP/s, 53 % of the fp32 matrix rate).
#include <stdio.h>
#include <type_traits>
#include "common.h"
#include "gemm_common.h"

namespace lp {

namespace {

constexpr int kMaxFGroup = 16;

// How an operand is read: element by element; k contiguous in whole 4-element loads; k-major in whole loads of T rows.
enum FMode { F_ANY, F_K4, F_ROWS };

template <typename T>
struct FProblem {
  const T* A; const T* B;
  int64_t lda, ldb;
  int a_kc, b_kc, a_mode, b_mode;    // see FMode
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

// Tile row that lane i's element of the t-th 16-row group is.
template <int MODE, int TT> __device__ __forceinline__ int tile_row(int t, int i) { return MODE == F_ROWS ? TT * i + t : 16 * t + i; }

// One lane's elements of a 16-deep chunk, k .. k + 3 of its TT rows.  p[t]: row t (F_ROWS: p[0], the first of TT neighbours).
// MASK: the chunk may reach past K (clamped for the load, zeroed after it).
template <int MODE, bool MASK, int TT, typename T>
__device__ __forceinline__ void fetch_chunk(const T* const (&p)[TT], int64_t st, int k, int K, f4 (&r)[TT]) {
  if constexpr (MODE == F_K4) {
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      r[t] = load4(p[t] + (MASK && k >= K ? K - 4 : k));
      if (MASK && k >= K) r[t] = f4{0.f, 0.f, 0.f, 0.f};
    }
  } else if constexpr (MODE == F_ROWS) {
    static_assert(TT == 4, "rows are read in fours");
    const T* q = p[0] + (int64_t)(MASK && k >= K ? K - 1 : k) * st;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f4 v = load4(q);
#pragma unroll
      for (int t = 0; t < TT; ++t) r[t][j] = !MASK || k + j < K ? v[t] : 0.f;
      if (!MASK || k + j + 1 < K) q += st;
    }
  } else {
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int kk = MASK ? (k + j < K ? k + j : K - 1) : k + j;
        const float v = to_f(p[t][kk * st]);
        r[t][j] = !MASK || k + j < K ? v : 0.f;
      }
  }
}

// The reduction of one wave: chunks c0 .. c1, DEPTH - 1 of them in flight.
template <int AM, int BM, int TT, int DEPTH, typename T>
__device__ __forceinline__ void reduce_wave(const T* const (&ap)[TT], const T* const (&bp)[TT], int64_t ast, int64_t bst, int g,
                                            int c0, int c1, int K, bool sums, f4 (&acc)[TT][TT], float (&rs)[TT]) {
  f4 a[DEPTH][TT], b[DEPTH][TT];
  auto fetch = [&](int s, int c) {
    const int k = 16 * c + 4 * g;
    if (16 * c + 16 <= K) {
      fetch_chunk<AM, false, TT>(ap, ast, k, K, a[s]);
      fetch_chunk<BM, false, TT>(bp, bst, k, K, b[s]);
    } else {
      fetch_chunk<AM, true, TT>(ap, ast, k, K, a[s]);
      fetch_chunk<BM, true, TT>(bp, bst, k, K, b[s]);
    }
  };
#pragma unroll
  for (int s = 0; s < DEPTH - 1; ++s)
    if (c0 + s < c1) fetch(s, c0 + s);
  for (int c = c0; c < c1; c += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {
      if (c + u >= c1) break;
      if (c + u + DEPTH - 1 < c1) fetch((u + DEPTH - 1) % DEPTH, c + u + DEPTH - 1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int x = 0; x < TT; ++x)
#pragma unroll
          for (int y = 0; y < TT; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][x][j], b[u][y][j], acc[x][y], 0, 0, 0);
      if (sums) {
#pragma unroll
        for (int x = 0; x < TT; ++x) rs[x] += (a[u][x][0] + a[u][x][1]) + (a[u][x][2] + a[u][x][3]);
      }
    }
  }
}

// A wave's partial tile and row sums into its part of LDS.  Accumulator v of lane (li, g) is row 4 g + v, column li of its
// 16 x 16 tile.
template <int AM, int BM, int TT>
__device__ __forceinline__ void leave_partial(const f4 (&acc)[TT][TT], float (&rs)[TT], bool sums, float* mine, float* rsum, int li, int g) {
  constexpr int EDGE = 16 * TT, LDP = EDGE + 4;
#pragma unroll
  for (int x = 0; x < TT; ++x)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      float* row = mine + tile_row<AM, TT>(x, 4 * g + v) * LDP;
      if constexpr (BM == F_ROWS && TT == 4) {
        *reinterpret_cast<f4*>(row + 4 * li) = f4{acc[x][0][v], acc[x][1][v], acc[x][2][v], acc[x][3][v]};
      } else {
#pragma unroll
        for (int y = 0; y < TT; ++y) row[tile_row<BM, TT>(y, li)] = acc[x][y][v];
      }
    }
  if (sums) {
#pragma unroll
    for (int x = 0; x < TT; ++x) {
      rs[x] += __shfl_xor(rs[x], 16, 64);
      rs[x] += __shfl_xor(rs[x], 32, 64);
      if (g == 0) rsum[tile_row<AM, TT>(x, li)] = rs[x];
    }
  }
}

template <typename T, int TT, int NP>
__global__ void __launch_bounds__(256, TT == 4 ? 2 : 1) k_gemm_f(FGroup<T, NP> grp) {
  constexpr int EDGE = 16 * TT, LDP = EDGE + 4;       // LDS rows of a partial tile
  constexpr int DEPTH = TT == 4 ? 3 : 4;       // chunks in registers
  extern __shared__ __attribute__((aligned(16))) float part[];      // [4][EDGE][LDP], then [4][EDGE] row sums
  int pi = 0;
#pragma unroll
  for (int i = 1; i < NP; ++i)
    if (i < grp.n && (int)blockIdx.x >= grp.p[i].first) pi = i;
  const FProblem<T>& P = grp.p[pi];
  const int tile = blockIdx.x - P.first, tm = tile / P.tiles_n, tn = tile - tm * P.tiles_n;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int K = P.K, nch = (K + 15) / 16;               // a wave's share of the reduction: whole chunks
  const int c0 = nch * wave / 4, c1 = nch * (wave + 1) / 4;
  const bool sums = P.rowsum && tn == 0;
  f4 acc[TT][TT];
  float rs[TT];
#pragma unroll
  for (int i = 0; i < TT; ++i) {
    rs[i] = 0.f;
#pragma unroll
    for (int j = 0; j < TT; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
  }
  const int64_t ast = P.a_kc ? 1 : P.lda, bst = P.b_kc ? 1 : P.ldb;
  auto rows = [&](auto mode, const T* base, bool kc, int64_t ld, int first, int n, const T* (&p)[TT]) {
    constexpr int MODE = decltype(mode)::value;
#pragma unroll
    for (int t = 0; t < TT; ++t) {
      int r = first + tile_row<MODE, TT>(t, li);
      const int last = MODE == F_ROWS ? n - TT + t : n - 1;       // whole loads of TT rows
      r = r < last ? r : last;
      p[t] = base + (kc ? (int64_t)r * ld : (int64_t)r);
    }
  };
  float* mine = part + (size_t)wave * EDGE * LDP;
  float* rsum = part + (size_t)4 * EDGE * LDP;
  // What the epilogue reads is asked for before the partial tiles are exchanged: element by element behind the reduction,
  // its loads were a chain of memory latencies longer than the product (16 elements a thread for a 64 x 64 tile: 20 us).
  // Thread: PER runs of W consecutive columns (64: 4 x 4, 32: 1 x 4, 16: 1 x 1).
  constexpr int W = TT == 1 ? 1 : 4, RUNS = EDGE * EDGE / W, PER = RUNS / 256, RPR = EDGE / W;     // runs per row
  const Epilogue& e = P.e;
  float eb[PER][W], es[PER][W], er[PER][W], ec[PER][W];
  auto ask = [&] {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int run = threadIdx.x + 256 * q;
      int m = tm * EDGE + run / RPR;
      m = m < P.M ? m : P.M - 1;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        int n = tn * EDGE + (run % RPR) * W + w;
        n = n < P.N ? n : P.N - 1;
        eb[q][w] = e.bias ? e.bias[n] : 0.f;
        es[q][w] = e.dact != ACT_NONE ? to_f(reinterpret_cast<const T*>(e.dact_src)[(size_t)m * e.ldd + n]) : 0.f;
        er[q][w] = e.res ? to_f(reinterpret_cast<const T*>(e.res)[(size_t)m * e.ldr + n]) : 0.f;
        const size_t o = (size_t)m * e.ldc + n;
        ec[q][w] = e.accumulate ? (e.c_f32 ? reinterpret_cast<const float*>(e.C)[o] : to_f(reinterpret_cast<const T*>(e.C)[o])) : 0.f;
      }
    }
  };
  typedef std::integral_constant<int, F_ANY> Any;
  typedef std::integral_constant<int, F_K4> K4;
  typedef std::integral_constant<int, TT == 4 ? F_ROWS : F_ANY> Rows;
  const T *ap[TT], *bp[TT];
  if constexpr (TT != 2) {
    auto product = [&](auto am, auto bm) {
      constexpr int AM = decltype(am)::value, BM = decltype(bm)::value;
      rows(am, P.A, P.a_kc, P.lda, tm * EDGE, P.M, ap);
      rows(bm, P.B, P.b_kc, P.ldb, tn * EDGE, P.N, bp);
      reduce_wave<AM, BM, TT, DEPTH>(ap, bp, ast, bst, g, c0, c1, K, sums, acc, rs);
      ask();
      leave_partial<AM, BM, TT>(acc, rs, sums, mine, rsum + wave * EDGE, li, g);
    };
    auto by_b = [&](auto am) {
      if (P.b_mode == F_K4) product(am, K4{});
      else if (TT == 4 && P.b_mode == F_ROWS) product(am, Rows{});
      else product(am, Any{});
    };
    if (P.a_mode == F_K4) by_b(K4{});
    else if (TT == 4 && P.a_mode == F_ROWS) by_b(Rows{});
    else by_b(Any{});
  } else {                 // 32-wide tiles: only the reduction's code is there in several forms (56.6 -> 55.4 us, two layers of 324)
    rows(Any{}, P.A, P.a_kc, P.lda, tm * EDGE, P.M, ap);
    rows(Any{}, P.B, P.b_kc, P.ldb, tn * EDGE, P.N, bp);
    if (P.a_mode == F_K4) {
      if (P.b_mode == F_K4) reduce_wave<F_K4, F_K4, TT, DEPTH>(ap, bp, ast, bst, g, c0, c1, K, sums, acc, rs);
      else reduce_wave<F_K4, F_ANY, TT, DEPTH>(ap, bp, ast, bst, g, c0, c1, K, sums, acc, rs);
    } else {
      if (P.b_mode == F_K4) reduce_wave<F_ANY, F_K4, TT, DEPTH>(ap, bp, ast, bst, g, c0, c1, K, sums, acc, rs);
      else reduce_wave<F_ANY, F_ANY, TT, DEPTH>(ap, bp, ast, bst, g, c0, c1, K, sums, acc, rs);
    }
    ask();
    leave_partial<F_ANY, F_ANY, TT>(acc, rs, sums, mine, rsum + wave * EDGE, li, g);
  }
  __syncthreads();
  constexpr int PT = EDGE * LDP;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int run = threadIdx.x + 256 * q, r = run / RPR, col = (run % RPR) * W, m = tm * EDGE + r;
    const float* p = part + r * LDP + col;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int n = tn * EDGE + col + w;
      float v = ((p[w] + p[PT + w]) + (p[2 * PT + w] + p[3 * PT + w])) + eb[q][w];
      if (m >= P.M || n >= P.N) continue;
      const size_t o = (size_t)m * e.ldc + n;
      if (e.pre) reinterpret_cast<T*>(e.pre)[o] = from_f<T>(v);
      if (e.act == ACT_RELU) v = fmaxf(v, 0.f);
      else if (e.act == ACT_GELU) v = gelu_f(v);
      if (e.dact == ACT_RELU) v = es[q][w] > 0.f ? v : 0.f;
      else if (e.dact == ACT_GELU) v *= dgelu_f(es[q][w]);
      v += er[q][w] + ec[q][w];
      if (e.c_f32) reinterpret_cast<float*>(e.C)[o] = v;
      else reinterpret_cast<T*>(e.C)[o] = from_f<T>(v);
    }
  }
  if (sums && (int)threadIdx.x < EDGE) {
    const int m = tm * EDGE + threadIdx.x;
    if (m < P.M) {
      const float* q = rsum + threadIdx.x;
      const float v = (q[0] + q[EDGE]) + (q[2 * EDGE] + q[3 * EDGE]);
      P.rowsum[m] = e.accumulate ? P.rowsum[m] + v : v;
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
  if (shm > 64 * 1024) {
    static LdsLimit limit;
    hipError_t e = limit.raise(reinterpret_cast<const void*>(k_gemm_f<T, TT, NP>), (int)shm);
    if (e != hipSuccess) return e;
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
    auto mode = [&](const void* base, int64_t ld, int kc, int n) {      // rows: whole loads of four
      if (ld % 4 || ((uintptr_t)base & al)) return F_ANY;
      return kc ? (g.K % 4 == 0 ? F_K4 : F_ANY) : (n % 4 == 0 ? F_ROWS : F_ANY);
    };
    p.a_mode = mode(g.A, g.lda, g.a_kc, g.M);
    p.b_mode = mode(g.B, g.ldb, g.b_kc, N);
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
  if (c.dt == BF16) {
    for (int i = 0; i < n; ++i) {
      hipError_t e = gemm_f_t<bf16_t, 1>(c, gs + i, 1);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  for (int i = 0; i < n; i += kMaxFGroup) {          // the table travels as a kernel argument: 1, 4 or 16 entries
    const int k = n - i < kMaxFGroup ? n - i : kMaxFGroup;
    hipError_t e = k == 1 ? gemm_f_t<float, 1>(c, gs + i, 1) : (k <= 4 ? gemm_f_t<float, 4>(c, gs + i, k) : gemm_f_t<float, kMaxFGroup>(c, gs + i, k));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lp
