// bf16 products on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation): which shapes they take, and the
// choice between the two kernels.
//
// One-tile-per-block kernel (kernels_gemm_tile.hip): every 8-aligned shape, six tile shapes from 64 x 64 to 256 x 256, long
// reductions over few tiles cut along k.
// Persistent kernel (kernels_gemm_dma.hip): large products, 256 x 256 tiles whose last partial wave is cut along k.
// In both the operand tiles go global -> LDS without passing registers.  An operand stored with the reduction index
// contiguous ("kc": forward activations and [out,in] weights) sits in LDS as [row][k] and is read with 16-byte ds_read; one
// stored with the reduction index as the slow dimension (dgrad weights, both wgrad operands) sits as [k][row], exactly as in
// memory, and is read with the gfx950 transposing LDS read (ds_read_b64_tr_b16), so nothing is ever transposed by the vector
// ALU.  The MFMA takes the n-side fragment as its first operand, which leaves each lane with runs of 8 consecutive n for one
// m: the fused epilogue (bias, activation, saved pre-activation, activation derivative, residual, accumulate) reads and
// writes 16 bytes per lane.
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#include "common.h"
#include "gemm_common.h"
#include "row_loss.h"

namespace lp {

hipError_t gemm_f32(const OpCtx& c, const GemmArgs* gs, int n);
bool gemm_dma_ok(const GemmArgs& g);
bool gemm_dma_plan(const OpCtx& c, const GemmArgs& g, int kind, int mode, DmaGemmPlan* out);
hipError_t gemm_dma(const OpCtx& c, const GemmArgs& g, const DmaGemmPlan& d);
bool gemm_dma_stats_ok(const GemmArgs& g, const DmaGemmPlan& d);
hipError_t gemm_dma_stats(const OpCtx& c, const GemmArgs& g, const DmaGemmPlan& d, const GroupStats& gs);
bool ce_fast_ok(const OpCtx& c, const void* z, int64_t ld, int n);
hipError_t ce_finish(const OpCtx& c, const GroupStats& g, float* loss_rows, int rows, int n);
hipError_t gemm_dma_grouped(const OpCtx& c, const GemmArgs* gs, int n);
TilePlan gemm_tile_plan(const OpCtx& c, const GemmArgs* gs, int n);
hipError_t gemm_tile(const OpCtx& c, const GemmArgs* gs, int n, const TilePlan& plan);

namespace {

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// Shapes the MFMA kernels take: every vector access must be 16-byte aligned and never straddle an edge.  The
// reduction may have any length where both operands are stored k-major (a weight gradient over any number of rows:
// a chunk lies along the rows of the tile, so K only counts chunks).  What they do not take runs in
// fp32 arithmetic; on the FMA kernel that it ran on before, with 2555 rows (K % 8 = 3) and a vocabulary of 10003 a step of six 448-wide layers took 18.1 ms, 16.3 of
// them in 27 plain products (a 1344 x 448 weight gradient 390 .. 660 us); 2.1 ms with them here.
bool fast_ok(const GemmArgs& g) {
  if (g.M < 1 || g.N < 8 || g.K < 1) return false;
  if (g.N % 8 || g.lda % 8 || g.ldb % 8 || g.ldc % 8) return false;
  if ((g.a_kc || g.b_kc) && g.K % 8) return false;
  if (!g.a_kc && (rows_of_a(g) % 8 || rows_of_a(g) < 8)) return false;
  if (!g.b_kc && (rows_of_b(g) % 8 || rows_of_b(g) < 8)) return false;
  if (!aligned16(g.A) || !aligned16(g.B) || !aligned16(g.C)) return false;
  if (g.bias && !aligned16(g.bias)) return false;
  if (g.pre && !aligned16(g.pre)) return false;
  if (g.dact_src && (!aligned16(g.dact_src) || g.ldd % 8)) return false;
  if (g.res && (!aligned16(g.res) || g.ldr % 8)) return false;
  return true;
}

}  // namespace

// Forced kernel: 0 none; 2 one tile per block; 3 + 2*kind + cut for the persistent kernel of tile shape
// `kind` (0: 256 x 128; 1: 256 x 256 with 8 waves; 2: 256 x 256 with 4 waves) with the tail whole (cut 0)
// or cut along k (cut 1); 9 + kind for that shape in panel mode; 13 + 2*kind for that shape with any of them.
// LP_GEMM_KERNEL = v2 | dma2 | dma4 | dmaw, optionally followed by w, c or p (dma4c, ...), forces one for a
// whole process (for measurements); a shape the forced kernel does not take falls back to the others.
static int env_choice() {
  static int v = -1;
  if (v < 0) {
    const char* s = getenv("LP_GEMM_KERNEL");
    v = 0;
    if (s && s[0] == 'v') v = 2;
    else if (s && s[0] == 'd' && s[1] == 'm' && s[2] == 'a') {
      const int kind = s[3] == '2' ? 0 : (s[3] == '4' ? 1 : (s[3] == 'w' ? 2 : -1));
      if (kind >= 0) v = s[4] == 'w' ? 3 + 2 * kind : (s[4] == 'c' ? 4 + 2 * kind : (s[4] == 'p' ? 9 + kind : 13 + 2 * kind));
    }
  }
  return v;
}

// A small cost model picks the kernel.  The persistent kernel's variants have a measured cost per k-step of one block and a
// fixed cost per tile (pipeline fill, epilogue); a cut adds the traffic of its fp32 partial sums and a second launch.  The
// other kernel prices its own shapes (gemm_tile_plan).
static const double kPartialBytesPerCycle = 4.0e12 / 2.4e9;   // partial sums: written, then read once more
static const double kSecondLaunchCycles = 12000.0;
static const double kCyclesPerUs = 2400.0, kDmaLaunchUs = 3.0;
static bool trace_on() {     // LP_GEMM_TRACE=1 prints the chosen kernel and plan of every GEMM (for measurements)
  static int v = -1;
  if (v < 0) { const char* s = getenv("LP_GEMM_TRACE"); v = (s && s[0] == '1') ? 1 : 0; }
  return v != 0;
}
// (8192 cubed, 32-deep 256 x 256: 854 us, 64-deep: 806.)
static const double kDmaStep[4] = {2796.0, 2050.0, 2050.0, 3900.0};      // 256 x 128 (two per CU), 256 x 256; 64-deep
static const double kDmaFixed[4] = {7000.0, 9000.0, 9000.0, 9000.0};
// Anything fused leaves this kernel's tiles in pieces of 16 bytes per lane, with its matrix cores idle: per tile, and once more
// for every matrix that the epilogue reads or writes beside the output.  8192 x 3072 x 768, 256 x 256 tiles / one tile per
// block: nothing fused 49 / 57 us, a bias 63 / 57, bias, GELU and pre-activation 78 / 63, residual 73 / 61; 8192 x 4096 x 1024
// 66 / 72, 77 / 72, 114 / 80, 94 / 80.  So a layer's products with K <= 1024 go one tile per block although their plain
// forms are faster here (all of them here: twelve layers of 768 25.2 -> 25.7 ms a step, 24 of 1024 34.9 -> 35.9).
static const double kDmaFused[4] = {10400.0, 15600.0, 15600.0, 15600.0};
// What a bf16 output takes at the rate it can leave at, in microseconds: the bound of short reductions over large outputs.  The
// 256-wide shapes write whole lines past L2 where nothing is fused and rows are whole lines (8192 x 32000 x 32: 110 us, 4.8 TB/s),
// and pieces of lines where they are not (8192 x 24008 x 32: 214 us); the others write pieces that L2 collects, up to the
// memory-side cache's 256 MB at 4.2 TB/s (8192 x 8000 x 32: 31 us), beyond it slower (8192 x 32000 x 32: 142 us; with a bias 220
// us, 203 us in 256-wide tiles).
static double store_us(const GemmArgs& g, int kind, bool fused) {
  if (g.c_f32) return 0.0;
  const double mb = 2e-6 * g.M * g.N;
  if (fused) return mb / (mb > 256.0 ? 2.5 : 4.2);
  if (kind == 0 || kind == 2) return mb / (mb > 256.0 ? 3.5 : 4.2);
  return mb / (g.ldc % 64 == 0 && ((uintptr_t)g.C & 127) == 0 ? 4.8 : 2.0);
}

static bool deep_auto() {     // LP_GEMM_K64=0 keeps the 64-deep k-tiles out of the automatic choice (for measurements)
  static int v = -1;
  if (v < 0) { const char* s = getenv("LP_GEMM_K64"); v = (s && s[0] == '0') ? 0 : 1; }
  return v != 0;
}

// Short reductions over at most two waves of tiles (a layer's K = 768 products): with anything fused they go one tile per block
// at these prices too, and plain ones are within a tenth of each other (8192 x 3072 x 768 49 us here, 57 one tile per block;
// 2184 x 6408 x 832 32 and 30, 980 x 31144 x 312 44 and 38), so the search over this kernel's plans, half a microsecond on the host, is left out.
static bool short_and_few(const GemmArgs& g) { return g.K <= 1024 && (long)((g.M + 255) / 256) * ((g.N + 255) / 256) <= 512; }

// The kernel and plan of a product; false where the kernel that is forced does not take it.
static bool choose(const OpCtx& c, const GemmArgs& g, bool* dma, DmaGemmPlan* dma_plan, TilePlan* tile_plan) {
  const int choice = c.gemm_variant ? c.gemm_variant : env_choice();
  double best = 1e300;
  // direct-to-LDS persistent kernel: tile shape x (tail whole, cut along k, panel mode)
  DmaGemmPlan best_dma;
  bool use_dma = false;
  int force_kind = -1, force_cut = -1;
  if (choice >= 20 && choice <= 22) { force_kind = 3; force_cut = choice - 20; }     // 64-deep k-tiles: tail whole / cut / panel mode
  else if (choice >= 13) force_kind = (choice - 13) / 2;
  else if (choice >= 9) { force_kind = choice - 9; force_cut = 2; }
  else if (choice >= 3) { force_kind = (choice - 3) / 2; force_cut = (choice - 3) % 2; }
  const int streams = (g.pre ? 1 : 0) + (g.dact != ACT_NONE ? 1 : 0) + (g.res ? 1 : 0) + (g.accumulate ? 1 : 0);
  const bool fused = streams || g.bias || g.act != ACT_NONE;
  if (gemm_dma_ok(g) && choice != 2 && !(choice == 0 && short_and_few(g))) {
    for (int kind = 0; kind < 4; ++kind) {
      if (force_kind >= 0 ? kind != force_kind : (kind == 2 || (kind == 3 && !deep_auto()))) continue;   // the 4-wave shape only when asked for
      for (int cut = 0; cut < 3; ++cut) {                 // tail whole / cut along k / panel mode
        if (force_cut >= 0 && cut != force_cut) continue;
        DmaGemmPlan d;
        if (!gemm_dma_plan(c, g, kind, cut, &d)) continue;
        if (cut == 1 && d.partial_bytes == 0 && force_cut < 0) continue;      // same as the uncut plan
        double cycles = d.steps * kDmaStep[kind] + d.items * (kDmaFixed[kind] + (fused ? (1 + streams) * kDmaFused[kind] : 0.0));
        const double store = kCyclesPerUs * store_us(g, kind, fused);
        if (store > cycles) cycles = store;
        if (d.partial_bytes > 0) cycles += 2.0 * d.partial_bytes / kPartialBytesPerCycle + kSecondLaunchCycles;
        // cut along k tile by tile, the tile columns of a row are at different k-steps and each fetches the
        // row's operand for itself: measured ~8 % slower than panel mode on a vocabulary head's gradients
        if (cut == 1 && d.partial_bytes > 0 && d.tiles_n >= 2 && d.tiles_n <= 8) cycles *= 1.12;
        if (cycles < best) { best = cycles; best_dma = d; use_dma = true; }
      }
    }
  }
  if (c.gemm_variant > 2 && !use_dma) return false;   // the forced kernel does not take this shape
  TilePlan tile;
  if (choice <= 2 || !use_dma) {
    tile = gemm_tile_plan(c, &g, 1);
    // a tenth in hand: at equal estimates the persistent kernel is ahead (8192 cubed 816 against 835 us, 32000 x 768 x 8192
    // 401 against 412)
    if (use_dma && 1.1 * tile.us < best / kCyclesPerUs + kDmaLaunchUs) use_dma = false;
  }
  if (trace_on())
    fprintf(stderr, "lp gemm %d x %d x %d (%d%d): %s %d full %d tail %d upb %d/%d sib %d pieces %d est %.1f us\n", g.M, g.N, g.K,
            g.a_kc, g.b_kc, use_dma ? "persistent, kind" : "tiles, shape", use_dma ? best_dma.kind : tile.shape,
            use_dma ? best_dma.full : 0, use_dma ? best_dma.tail_tiles : 0, use_dma ? best_dma.upb : 0,
            use_dma ? best_dma.kt : 0, use_dma ? best_dma.sib : 0, use_dma ? 1 : tile.splits,
            use_dma ? best / kCyclesPerUs + kDmaLaunchUs : tile.us);
  *dma = use_dma; *dma_plan = best_dma; *tile_plan = tile;
  return true;
}

hipError_t gemm_mfma(const OpCtx& c, const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  bool dma;
  DmaGemmPlan d;
  TilePlan t;
  if (!choose(c, g, &dma, &d, &t)) return hipErrorInvalidValue;
  return dma ? gemm_dma(c, g, d) : gemm_tile(c, &g, 1, t);
}

static int use_plain() {
  static int v = -1;
  if (v < 0) { const char* s = getenv("LP_PLAIN_GEMM"); v = (s && s[0] == '1') ? 1 : 0; }
  return v;
}

hipError_t op_gemm(const OpCtx& c, const GemmArgs& g) {
  const uint64_t tag = (uint64_t)(g.M & 0xfffff) | (uint64_t)(g.N & 0xfffff) << 20 | (uint64_t)(g.K & 0xfffff) << 40 |
                       (uint64_t)(g.a_kc != 0) << 60 | (uint64_t)(g.b_kc != 0) << 61 | (uint64_t)(g.c_f32 != 0) << 62;
  ProfScope prof_(c, KC_GEMM, 2.0 * g.M * g.N * g.K, tag);
  if (c.gemm_variant >= 2 && !(c.dt == BF16 && fast_ok(g))) return hipErrorInvalidValue;
  if (c.dt == BF16 && !use_plain() && fast_ok(g)) {
    if (g.rowsum) {            // the bf16 kernels take no row sums
      hipError_t e = op_colsum(c, g.A, g.lda, g.rowsum, g.K, g.M, g.accumulate);
      if (e != hipSuccess) return e;
    }
    return gemm_mfma(c, g);
  }
  return gemm_f32(c, &g, 1);
}

static bool grouping_off() {     // LP_NO_GROUP=1: every product in a launch of its own (for measurements)
  static int v = -1;
  if (v < 0) { const char* s = getenv("LP_NO_GROUP"); v = (s && s[0] == '1') ? 1 : 0; }
  return v != 0;
}

bool gemm_joins(const OpCtx& c, const GemmArgs* group, int n, const GemmArgs& g) {
  if (c.dt != BF16 || use_plain() || grouping_off() || env_choice() != 0 || c.gemm_variant != 0 || n >= kTileGroupMax || !fast_ok(g)) return false;
  GemmArgs all[kTileGroupMax];
  for (int i = 0; i < n; ++i) {
    if (!fast_ok(group[i]) || group[i].K != g.K || group[i].a_kc != g.a_kc || group[i].b_kc != g.b_kc) return false;
    all[i] = group[i];
  }
  all[n] = g;
  bool dma;
  DmaGemmPlan d;
  TilePlan alone;
  if (!choose(c, g, &dma, &d, &alone) || dma) return false;
  return gemm_tile_plan(c, all, n + 1).us < gemm_tile_plan(c, group, n).us + alone.us;
}

// The row losses of a head whose logits nothing else needs: instead of storing them (bf16 [rows, ld] into g.C) and reading them
// again, the product leaves a pair per row and 64 columns in that memory, a 16th of it (and the label's logit per row), and a
// short launch the losses; the bits of op_softmax_ce.  Only where the product itself would be uncut 256 x 256 tiles (a large
// head); hipErrorInvalidValue, with nothing launched, where not.  Twelve layers of 768, 8192 rows, 32000 classes: 8.66 -> 7.72 ms
// an evaluation.
static bool loss_plan(const OpCtx& c, const GemmArgs& g, DmaGemmPlan* d) {
  if (c.dt != BF16 || use_plain() || !fast_ok(g) || !ce_fast_ok(c, g.C, g.ldc, g.N)) return false;
  if (g.bias || g.pre || g.act != ACT_NONE || g.dact != ACT_NONE || g.res || g.accumulate || g.c_f32 || g.rowsum) return false;
  if (((size_t)8 * ((g.N + 63) / 64) + 4) > (size_t)2 * g.ldc) return false;
  if (c.gemm_variant == 0 && env_choice() == 0 && short_and_few(g)) return false;      // without pricing it: small evaluations wait for the host
  bool dma;
  TilePlan t;
  return choose(c, g, &dma, d, &t) && dma && gemm_dma_stats_ok(g, *d);
}
bool gemm_loss_ok(const OpCtx& c, const GemmArgs& g) { DmaGemmPlan d; return loss_plan(c, g, &d); }
hipError_t op_gemm_loss(const OpCtx& c, const GemmArgs& g, const int32_t* y, float* loss_rows) {
  DmaGemmPlan d;
  if (!loss_plan(c, g, &d)) return hipErrorInvalidValue;
  GroupStats gs;
  gs.groups = (g.N + 63) / 64; gs.y = y;
  gs.pair = (float2*)g.C; gs.zy = (float*)(gs.pair + (size_t)g.M * gs.groups);
  ProfScope prof_(c, KC_GEMM, 2.0 * g.M * g.N * g.K);
  hipError_t e = gemm_dma_stats(c, g, d, gs);
  return e == hipSuccess ? ce_finish(c, gs, loss_rows, g.M, g.N) : e;
}

// n <= kTileGroupMax products in one launch of the one-tile-per-block kernel, whatever the other grouped kernel would cost.
hipError_t gemm_tile_grouped(const OpCtx& c, const GemmArgs* gs, int n) {
  if (n < 1 || n > (c.with_sums ? kTileGroupMax : 4) || c.dt != BF16) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (!fast_ok(gs[i]) || gs[i].K != gs[0].K || gs[i].a_kc != gs[0].a_kc || gs[i].b_kc != gs[0].b_kc || (gs[i].rowsum && !c.with_sums)) return hipErrorInvalidValue;
  return gemm_tile(c, gs, n, gemm_tile_plan(c, gs, n));
}

hipError_t op_gemm_grouped(const OpCtx& c, const GemmArgs* gs, int n) {
  if (c.dt == F32 && n >= 2) {
    double flops = 0.0;
    for (int i = 0; i < n; ++i) flops += 2.0 * gs[i].M * gs[i].N * gs[i].K;
    ProfScope prof_(c, KC_GEMM, flops);
    return gemm_f32(c, gs, n);
  }
  if (n >= 2 && c.dt == BF16 && !use_plain() && !grouping_off() && c.gemm_variant == 0 && env_choice() == 0) {
    bool ok = true;
    for (int i = 0; i < n; ++i) ok = ok && fast_ok(gs[i]);
    if (ok) {
      // Up to four products of one reduction length and layout (a layer's weight gradients) share a launch of the tile kernel,
      // alone against the persistent group and its fix-up: width 768 over 8192 rows 116 and 152 us, 1024 201 and 238, 448 over
      // 2555 24 and 43; level where the work is largest (768 over 32768 rows 455 and 465, 2048 over 8192 703 and 714).  More of them,
      // or unequal ones, go to that kernel.
      bool tiles = n <= 4 || (n <= kTileGroupMax && c.with_sums);
      double flops = 0.0;
      for (int i = 0; i < n; ++i) {
        const GemmArgs& g = gs[i];
        tiles = tiles && g.K == gs[0].K && g.a_kc == gs[0].a_kc && g.b_kc == gs[0].b_kc && (!g.rowsum || (c.with_sums && !g.a_kc && !g.b_kc));
        flops += 2.0 * g.M * g.N * g.K;
      }
      TilePlan plan;
      if (tiles) plan = gemm_tile_plan(c, gs, n);
      if (plan.shape >= 0) {
        ProfScope prof_(c, KC_GEMM, flops);
        return gemm_tile(c, gs, n, plan);
      }
      if (!c.with_sums) {
        hipError_t e = gemm_dma_grouped(c, gs, n);
        if (e != hipErrorInvalidValue) return e;        // launched (or failed for a reason of the device's)
      }
    }
  }
  if (c.with_sums) {                   // the sums by themselves, then the products
    std::vector<const void*> dy;
    std::vector<GemmArgs> plain(gs, gs + n);
    std::vector<int64_t> ld;
    std::vector<float*> out;
    std::vector<int> m;
    for (GemmArgs& g : plain) {
      if (!g.rowsum) continue;
      dy.push_back(g.A); ld.push_back(g.lda); out.push_back(g.rowsum); m.push_back(g.M);
      g.rowsum = nullptr;
    }
    hipError_t e = op_colsum_batched(c, (int)out.size(), dy.data(), ld.data(), out.data(), gs[0].K, m.data(), gs[0].accumulate);
    if (e == hipSuccess) e = op_add_pending(c);
    OpCtx o = c;
    o.with_sums = false;
    return e == hipSuccess ? op_gemm_grouped(o, plain.data(), n) : e;
  }
  for (int i = 0; i < n; ++i) {
    hipError_t e = op_gemm(c, gs[i]);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace lp
