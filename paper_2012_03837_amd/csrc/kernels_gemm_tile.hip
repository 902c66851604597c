// bf16 products with one output tile per block (gemm_tile.h): every aligned shape that is too small or too odd for the
// persistent kernel (kernels_gemm_dma.hip), one product or up to four of one reduction length and layout in a launch.
//
// What bounds it.  A tile of BM x BN takes BM x BN / 32 clocks of a compute unit's matrix cores per 64 of k, and
// (BM + BN) x 2 clocks of its 64 byte / clock path from L2: 128 x 128 spends as long on either, 256 x 256 half as long on
// the loads.  So large products want large tiles, and small ones as many tiles as there are compute units: with few tiles a
// product is the latency of its loads, which are all in flight at once up to 4 x 64 of k.  Tile shapes, measured alone
// (us; k contiguous in both operands):
//                        600 x 384 x 128   2555 x 1344 x 448   2048 x 512 x 2048   8192 x 768 x 3072   8192 x 4096 x 1024
//   64 x 64, 4 stages          3.8              12.5                 12.2               74.1               144
//   128 x 64, 3 stages         4.7               9.8                 15.2               62.3               136
//   128 x 128, 2 stages        6.1              10.6                 25.6               55.9               110
//   128 x 128, 4 stages        6.4              10.6                 19.4               62.7               145
//   256 x 128, 3 stages        7.2              12.2                 25.8               51.4               103
//   256 x 256, 2 stages       10.9              18.0                 45.7               76.2                91
// (the last with GELU and a stored pre-activation; 69 us without, where a kernel that staged its tiles through registers had 81,
// and 58.9, 16.3 + 5.3, 13 to 15 and 8.8 us on the others from the right).
#include <stdio.h>
#include "gemm_tile.h"
#include "pending.h"

namespace lp {

using namespace tile;

namespace {

constexpr int kTileGroup = kTileGroupMax;
struct TileProblem {
  Operand A, B;
  Epilogue e;
  int M, N, tiles_m, tiles_n;
  int first;             // number of its first tile
  size_t ws;             // offset of its partial sums, [splits][M][N], and of its row sums', [splits][M]
  size_t sum_ws;
  float* rowsum;         // rowsum[m] (+)= sum_k A(m, k) (null: not wanted)
};
template <int NP>
struct TileGroup { TileProblem p[NP]; int n, K, splits, per, tiles; float* ws; PendingTable pend; };   // per: k-tiles of a piece
template <>
struct TileGroup<1> { TileProblem p[1]; int n, K, splits, per, tiles; float* ws; };

template <bool A_KC, bool B_KC, int WGM, int WGN, int TM, int TN, int NST, int NP>
__global__ void __launch_bounds__(64 * WGM * WGN, WGM * WGN == 8 || (Shape<WGM, WGN, TM, TN, NST>::LDS <= 80 * 1024) ? 2 : 1)
k_gemm_tile(TileGroup<NP> g) {
  typedef Shape<WGM, WGN, TM, TN, NST> SH;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // A layer's weight gradients (both operands k-major) take its bias gradients along, as sums of A's rows in the blocks of the
  // first tile column, and its pending sums, in blocks behind the tiles: two launches fewer a layer, and dY is not read again.
  // Steps with a column-sum and an adding launch a layer / with both here: three layers of 128 over 600 rows 386 / 359 us, six
  // of 448 over 2555 1541 / 1483, 24 of 1024 over 8192 34.43 / 33.99 ms.
  constexpr bool SUMS = !A_KC && !B_KC && NP > 1;
  const int blocks = g.tiles * g.splits;
  if constexpr (SUMS) {
    if ((int)blockIdx.x >= blocks) {
      add_pending_block<WGM * WGN>(g.pend, blockIdx.x - blocks, reinterpret_cast<float (*)[64]>(smem));
      return;
    }
  }
  int q = xcd_range(blockIdx.x, blocks);
  const int piece = q / g.tiles;       // pieces of one k range are neighbours: they share operand panels in L2
  q -= piece * g.tiles;
  int pi = 0;
#pragma unroll
  for (int i = 1; i < NP; ++i)
    if (i < g.n && q >= g.p[i].first) pi = i;
  const TileProblem& P = g.p[pi];
  int tm, tn;
  tile_coords(q - P.first, P.tiles_m, P.tiles_n, tm, tn);
  const int nt = (g.K + KT - 1) / KT, t0 = piece * g.per, t1 = t0 + g.per < nt ? t0 + g.per : nt;
  const int mb = tm * SH::BM + (wave / WGN) * 32 * TM, nb = tn * SH::BN + (wave % WGN) * 32 * TN;
  const int M = P.M, N = P.N;
  const Epilogue e = P.e;
  const bool raw = g.splits > 1;
  f32x16 acc[TN][TM];
  RowStore<TM, TN> out;
  const DenseLoader<A_KC> la{P.A};
  const DenseLoader<B_KC> lb{P.B};
  typename std::conditional<SUMS, RowSums<TM>, NoTap>::type sums;
  if constexpr (SUMS) {
    sums.mask = 0;
    if (P.rowsum && tn == 0)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) sums.mask |= (kk % WGN == wave % WGN) << kk;
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int x = 0; x < RowSums<TM>::CH; ++x) sums.s[x][j] = 0.f;
  }
  multiply<SH, WGN, TM, TN, NST>(la, lb, tm * SH::BM, tn * SH::BN, t0, t1, g.K, smem, acc,
                                 [&] { if (!raw) out.prefetch(e, mb, nb, M, N, lane); }, sums);
  __syncthreads();                     // the stages become the waves' patches
  if constexpr (SUMS) {
    if (sums.mask) {                   // the waves' shares, added in wave order
      float* mine = reinterpret_cast<float*>(smem + wave * SH::PATCH);
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        float v = sums.s[0][j];
        if (RowSums<TM>::CH > 1) v += sums.s[RowSums<TM>::CH - 1][j];
        v += __shfl_xor(v, 32, 64);
        if (lane < 32) mine[32 * j + lane] = v;
      }
      __syncthreads();
      if (wave % WGN == 0) {
        for (int r = lane; r < 32 * TM; r += 64) {
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < WGN; ++w) v += mine[w * (SH::PATCH / 4) + r];
          const int m = mb + r;
          if (m >= M) continue;
          if (raw) g.ws[P.sum_ws + (size_t)piece * M + m] = v;
          else P.rowsum[m] = e.accumulate ? P.rowsum[m] + v : v;
        }
      }
      __syncthreads();
    }
  }
  ColumnSums<TN> none;
  out.template store<false>(e, acc, smem + wave * SH::PATCH, mb, nb, M, N, lane, raw ? g.ws + P.ws + (size_t)piece * M * N : nullptr,
                            none);
}

// Adds the pieces' partial sums in order and applies the epilogue; one thread per 8 columns, the problems one after the
// other in the grid.
template <int NP>
__global__ void __launch_bounds__(256) k_tile_reduce(TileGroup<NP> g) {
  size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  int pi = 0;
#pragma unroll
  for (int i = 0; i < NP - 1; ++i) {
    const size_t w = (size_t)g.p[i].M * (g.p[i].N >> 3);
    if (pi == i && i + 1 < g.n && idx >= w) { idx -= w; pi = i + 1; }
  }
  const TileProblem& P = g.p[pi];
  const int n8 = P.N >> 3;
  if (idx >= (size_t)P.M * n8) return;
  const int m = (int)(idx / n8), n = (int)(idx % n8) * 8;
  const size_t slab = (size_t)P.M * P.N;
  const float* src = g.ws + P.ws + (size_t)m * P.N + n;
  add_pieces(src, slab, g.splits, [&](float* v) { epilogue8(P.e, m, n, v); });
  if (NP > 1 && n == 0 && P.rowsum) {
    const float* sp = g.ws + P.sum_ws + m;
    float v = 0.f;
    int s = 0;
    for (; s + 8 <= g.splits; s += 8) {
      float a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = sp[(size_t)(s + u) * P.M];
#pragma unroll
      for (int u = 0; u < 8; ++u) v += a[u];
    }
    for (; s < g.splits; ++s) v += sp[(size_t)s * P.M];
    P.rowsum[m] = P.e.accumulate ? P.rowsum[m] + v : v;
  }
}

// Cost of a launch in microseconds: `fixed` (launch, first loads, epilogue), then per 64 of k `alone` where a compute unit has
// one block and `full` where it has as many as fit, `round` more for every round of blocks.
struct TileShape { int bm, bn, per_cu; double fixed, alone, full, round; };
const TileShape kShapes[kTileShapes] = {
    {64, 64, 2, 3.3, 0.27, 0.40, 1.8},   {128, 64, 2, 4.0, 0.30, 0.64, 3.1},  {128, 128, 2, 5.5, 0.52, 1.05, 5.7},
    {128, 128, 1, 5.8, 0.38, 0.70, 3.9}, {256, 128, 1, 6.0, 0.80, 0.95, 5.4}, {256, 256, 1, 8.0, 1.50, 1.62, 8.3},
    {64, 128, 2, 4.0, 0.30, 0.64, 3.1},  {256, 64, 2, 9.0, 0.60, 1.10, 5.0},       // convolutions only
    {128, 32, 4, 3.5, 0.25, 0.80, 2.0},
};

template <bool A_KC, bool B_KC, int WGM, int WGN, int TM, int TN, int NST, int NP>
hipError_t launch_shape(const OpCtx& c, const TileGroup<NP>& g, double flops) {
  typedef Shape<WGM, WGN, TM, TN, NST> SH;
  if (SH::LDS > 64 * 1024) {
    static LdsLimit limit;
    hipError_t e = limit.raise(reinterpret_cast<const void*>(k_gemm_tile<A_KC, B_KC, WGM, WGN, TM, TN, NST, NP>), SH::LDS);
    if (e != hipSuccess) return e;
  }
  static char name[80];
  if (!name[0])
    snprintf(name, sizeof name, "k_gemm_tile<%s, %s, %d, %d, %d, %d, %d, %d>", A_KC ? "true" : "false", B_KC ? "true" : "false", WGM,
             WGN, TM, TN, NST, NP);
  ProfScope one_(c, KC_GEMM_KERNEL, flops, 0, name);
  int blocks = g.tiles * g.splits;
  if constexpr (NP > 1) blocks += g.pend.blocks;
  k_gemm_tile<A_KC, B_KC, WGM, WGN, TM, TN, NST, NP><<<blocks, SH::THREADS, SH::LDS, c.stream>>>(g);
  return hipGetLastError();
}

template <bool A_KC, bool B_KC, int NP>
hipError_t launch_layout(const OpCtx& c, const TileGroup<NP>& g, int shape, double flops) {
  switch (shape) {
    case 0: return launch_shape<A_KC, B_KC, 2, 2, 1, 1, 4, NP>(c, g, flops);
    case 1: return launch_shape<A_KC, B_KC, 2, 2, 2, 1, 3, NP>(c, g, flops);
    case 2: return launch_shape<A_KC, B_KC, 2, 2, 2, 2, 2, NP>(c, g, flops);
    case 3: return launch_shape<A_KC, B_KC, 2, 2, 2, 2, 4, NP>(c, g, flops);
    case 4: return launch_shape<A_KC, B_KC, 4, 2, 2, 2, 3, NP>(c, g, flops);
    case 5: return launch_shape<A_KC, B_KC, 2, 4, 4, 2, 2, NP>(c, g, flops);
  }
  return hipErrorInvalidValue;
}

template <int NP>
hipError_t launch_group(const OpCtx& c, const GemmArgs* gs, int n, const TilePlan& plan) {
  const TileShape& s = kShapes[plan.shape];
  TileGroup<NP> g = {};
  g.K = gs[0].K; g.splits = plan.splits; g.per = plan.per; g.ws = c.splitk_ws;
  size_t ws = 0, work = 0;
  double flops = 0.0;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& a = gs[i];
    TileProblem& p = g.p[g.n++];
    p.A = Operand{(const bf16_t*)a.A, a.lda, rows_of_a(a)};
    p.B = Operand{(const bf16_t*)a.B, a.ldb, rows_of_b(a)};
    p.e = make_epilogue(a);
    p.M = a.M; p.N = a.N;
    p.tiles_m = (a.M + s.bm - 1) / s.bm; p.tiles_n = (a.N + s.bn - 1) / s.bn;
    p.first = g.tiles;
    g.tiles += p.tiles_m * p.tiles_n;
    p.ws = ws;
    ws += (size_t)plan.splits * a.M * a.N;
    work += (size_t)a.M * (a.N >> 3);
    flops += 2.0 * a.M * a.N * a.K;
  }
  if constexpr (NP > 1) {
    for (int i = 0; i < n; ++i) {
      g.p[i].rowsum = gs[i].rowsum;
      g.p[i].sum_ws = ws;
      if (gs[i].rowsum) ws += (size_t)plan.splits * gs[i].M;
    }
  }
  if (plan.splits > 1 && (!c.splitk_ws || ws > c.splitk_elems)) return hipErrorInvalidValue;
  const GemmArgs& a = gs[0];
  if constexpr (NP > 1)
    if (c.with_sums && !a.a_kc && !a.b_kc) g.pend = take_pending(c.pending);
  hipError_t e;
  if (a.a_kc && a.b_kc) e = launch_layout<true, true, NP>(c, g, plan.shape, flops);
  else if (a.a_kc) e = launch_layout<true, false, NP>(c, g, plan.shape, flops);
  else if (a.b_kc) e = launch_layout<false, true, NP>(c, g, plan.shape, flops);
  else e = launch_layout<false, false, NP>(c, g, plan.shape, flops);
  if (e != hipSuccess || plan.splits == 1) return e;
  k_tile_reduce<NP><<<(unsigned)((work + 255) / 256), 256, 0, c.stream>>>(g);
  return hipGetLastError();
}

}  // namespace

// The cheapest tile shape and number of pieces for n products that share a launch.  Long reductions over few tiles are cut
// into pieces of about eight k-tiles or more (the last may be shorter: 25 in three are 9, 9 and 7), whose fp32 partial sums a second launch adds in order (4.5 TB/s and 4.6 us: what the
// smallest launch costs behind another one).
TilePlan tile_plan(const OpCtx& c, int n, const int* M, const int* N, int K, unsigned mask, int max_pieces) {
  TilePlan best;
  const int nt = (K + KT - 1) / KT;
  if (c.tile_shape >= 0) {              // forced (nothing that the workspace does not hold)
    double elems = 0.0;
    for (int i = 0; i < n; ++i) elems += (double)M[i] * N[i];
    const int sp = c.tile_pieces < 1 ? 1 : c.tile_pieces, per = (nt + sp - 1) / sp, pieces = per > 0 ? (nt + per - 1) / per : 1;
    if (c.tile_shape >= kTileShapes || !(mask >> c.tile_shape & 1) || pieces != sp ||
        (pieces > 1 && (!c.splitk_ws || pieces * elems > (double)c.splitk_elems)))
      return best;
    best.shape = c.tile_shape; best.splits = pieces; best.per = per; best.us = 0.0;
    return best;
  }
  for (int s = 0; s < kTileShapes; ++s) {
    if (!(mask >> s & 1)) continue;
    const TileShape& h = kShapes[s];
    long tiles = 0;
    double elems = 0.0;
    for (int i = 0; i < n; ++i) {
      tiles += (long)((M[i] + h.bm - 1) / h.bm) * ((N[i] + h.bn - 1) / h.bn);
      elems += (double)M[i] * N[i];
    }
    if (tiles > (1L << 28)) continue;
    int last = -1;
    for (int sp = 1; sp <= max_pieces; ++sp) {
      if (sp > 1 && (!c.splitk_ws || nt < 8 * sp || sp * elems > (double)c.splitk_elems)) break;
      const int per = (nt + sp - 1) / sp;
      if (per == last) continue;
      last = per;
      const int pieces = per > 0 ? (nt + per - 1) / per : 1;          // no piece is empty
      const long blocks = tiles * pieces, slots = 256L * h.per_cu;
      double us = h.fixed;
      if (blocks <= 256) {
        us += per * h.alone;
      } else if (blocks <= slots) {      // one round, however full (528 x 11648 x 112 in 455 of 512 blocks: 10.5 us, 256 x 256 13.6)
        us += per * h.full + 0.5 * h.round;
      } else {
        const long rem = blocks % slots;
        us += (double)(blocks / slots) * (per * h.full + h.round);
        if (rem > 224 * h.per_cu) us += per * h.full + h.round;
        else if (rem > 0) us += per * (rem > 256 ? h.full : h.alone) + 0.5 * h.round;
      }
      if (pieces > 1) us += 4.6 + (pieces + 1) * elems * 4.0 / 4.5e6;
      if (us < best.us) { best.us = us; best.shape = s; best.splits = pieces; best.per = per; }
    }
  }
  return best;
}
TilePlan gemm_tile_plan(const OpCtx& c, const GemmArgs* gs, int n) {
  int M[kTileGroup], N[kTileGroup];
  constexpr int kPieces = 32;
  OpCtx o = c;
  for (int i = 0; i < n; ++i) {
    M[i] = gs[i].M; N[i] = gs[i].N;
    const size_t sums = gs[i].rowsum ? (size_t)kPieces * M[i] : 0;       // the row sums' part of the workspace
    o.splitk_elems = o.splitk_elems > sums ? o.splitk_elems - sums : 0;
  }
  return tile_plan(o, n, M, N, gs[0].K, 0x3f, kPieces);
}

// n products (one, or up to kTileGroupMax of one reduction length and the same operand layouts), all of shapes that the
// bf16 kernels take.
hipError_t gemm_tile(const OpCtx& c, const GemmArgs* gs, int n, const TilePlan& plan) {
  if (plan.shape < 0 || n < 1 || n > kTileGroup) return hipErrorInvalidValue;
  return n == 1 ? launch_group<1>(c, gs, 1, plan) : launch_group<kTileGroup>(c, gs, n, plan);
}

}  // namespace lp
