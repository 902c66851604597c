// bf16 product tile on the matrix cores, one output tile per block (and pieces that the persistent kernel shares): operand
// tiles stream global -> LDS with the 16-byte direct-to-LDS load through a ring of NST stages of 64 k, so that a short reduction is in flight as a whole and a long
// one NST - 1 k-tiles ahead.  Generic over the operands' loaders (dense matrices here, pixels in the convolutions).
//
// Block: WGM x WGN waves of (32 TM) x (32 TN), v_mfma_f32_32x32x16_bf16, the n-side fragment as the first operand.
// LDS tiles are unpadded (a direct-to-LDS load fills 1 KB of contiguous LDS per wave) with an XOR swizzle that each lane's
// global address undoes:
//   k contiguous: [row][8 chunks of 8 k], 128-byte rows, chunk c of row r in slot c ^ ((r >> 1) & 7)
//   k-major     : [64 k][ROWS / 8 chunks of 8 rows], chunk j of k-row k in slot j ^ kswz(k), read with ds_read_b64_tr_b16
// A chunk that does not exist (past the reduction's end, a convolution's padding) is loaded from a zero page.
#pragma once
#include "common.h"
#include "gemm_common.h"

namespace lp {
namespace tile {

constexpr int KT = 64;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

struct Operand { const bf16_t* p; int64_t ld; int rows; };

// MFMA row i of the n-side fragment holds tile column 16*(g/2) + 8*h + 4*(g%2) + j, i = 8g + 4h + j, so
// that accumulator values 0..7 / 8..15 of lane-half h are columns 8h..8h+7 / 16+8h..16+8h+7.
__device__ __forceinline__ int nmap(int i) {
  int g = i >> 3, h = (i >> 2) & 1, j = i & 3;
  return 16 * (g >> 1) + 8 * h + 4 * (g & 1) + j;
}

static __device__ const __attribute__((aligned(16))) unsigned kZeroPage[4] = {0, 0, 0, 0};

// 16 bytes per lane, global -> LDS, lane l's at dst + 16 l.  In assembly because of what the compiler does around the
// builtin: it knows that the load writes LDS, not where, and puts an s_waitcnt vmcnt(0) in front of the next
// ds_read_b64_tr_b16, so that a loop with a k-major operand never had a load in flight behind its matrix instructions
// (persistent kernel, both operands k-major, alone: 32000 x 768 x 8192 449 -> 401 us, 8192 cubed 964 -> 851 us; a layer's
// four weight gradients 159 -> 140 us at width 768, 256 -> 240 us at 1024).  Nothing is returned in registers; who reads the
// LDS waits with a barrier that clobbers memory.  m0 is a reserved register: the clobber draws a warning and protects nothing,
// but no other instruction of these kernels uses it (LDS instructions do not need it, and nothing is indexed by a register).
__device__ __forceinline__ void to_lds(const bf16_t* src, char* dst) {
  const unsigned at = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)dst;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(at), "v"(src) : "m0");
}

// k-major tiles: four neighbouring k-rows, which a transposing read takes together, in different quarters of the banks.
template <int ROWS>
__device__ __forceinline__ int kswz(int k) { return ROWS == 32 ? 0 : (ROWS == 64 ? ((k >> 1) & 1) << 2 : (k & 3) << 2); }

// Which chunk of a tile lane `lane` carries in the q-th 1 KB of it: (row, k) of its first element.
template <bool KC, int ROWS>
__device__ __forceinline__ void chunk_of(int q, int lane, int& row, int& k) {
  if (KC) {
    row = q * 8 + (lane >> 3);
    k = 8 * ((lane & 7) ^ ((row >> 1) & 7));
  } else {
    constexpr int CPR = ROWS / 8, KPI = 64 / CPR;      // chunks per k-row, k-rows per 1 KB
    k = q * KPI + lane / CPR;
    row = 8 * ((lane % CPR) ^ kswz<ROWS>(k));
  }
}

// A dense matrix.  Rows past the end are read from the last ones (their products are not stored).
template <bool KC_>
struct DenseLoader {
  static constexpr bool KC = KC_;
  Operand o;
  template <int ROWS, int NI>
  struct State {
    const bf16_t* g[NI];
    int64_t step;
  };
  template <int ROWS, int NI>
  __device__ __forceinline__ void init(State<ROWS, NI>& s, int r0, int q0, int lane, int k0) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int row, k;
      chunk_of<KC, ROWS>(q0 + i, lane, row, k);
      row += r0;
      if (KC) {
        row = row < o.rows ? row : o.rows - 1;
        s.g[i] = o.p + (size_t)row * o.ld + k0 + k;
      } else {
        row = row + 8 <= o.rows ? row : o.rows - 8;
        s.g[i] = o.p + (size_t)(k0 + k) * o.ld + row;
      }
    }
    s.step = KC ? KT : KT * o.ld;
  }
  // Load i of a k-tile (the caller asks for the loads of a k-tile in order).  PARTIAL: the k-tile may reach past K.
  template <bool PARTIAL, int ROWS, int NI>
  __device__ __forceinline__ void issue(State<ROWS, NI>& s, int i, char* dst, int q0, int lane, int kt, int K) const {
    const bf16_t* src = s.g[i];
    if (PARTIAL) {
      int row, k;
      chunk_of<KC, ROWS>(q0 + i, lane, row, k);
      if (kt * KT + k >= K) src = reinterpret_cast<const bf16_t*>(kZeroPage);
    }
    to_lds(src, dst + (q0 + i) * 1024);
    s.g[i] += s.step;
  }
};

// fragments of one 16-deep substep kk
__device__ __forceinline__ bf16x8 frag_kc(const char* sm, int row, int chunk) {
  return *reinterpret_cast<const bf16x8*>(sm + row * 128 + 16 * (chunk ^ ((row >> 1) & 7)));
}
template <int ROWS>
__device__ __forceinline__ bf16x8 frag_t(const char* sm, int rowbase, int k) {
  const char* p = sm + k * (ROWS * 2) + 16 * ((rowbase >> 3) ^ kswz<ROWS>(k)) + (rowbase & 7) * 2;
  bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p));
  bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 4 * ROWS * 2));
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) { r[e] = lo[e]; r[4 + e] = hi[e]; }
  return r;
}

// At most VM of this wave's vector-memory operations outstanding, its LDS reads done, then the barrier (one statement: the
// compiler neither moves LDS accesses across it nor makes it wait for every load).
template <int VM>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(VM) : "memory");
}

// Loads in part p of n loads in `parts` parts.
constexpr int part_of(int n, int parts, int p) { return (p + 1) * n / parts - p * n / parts; }

template <int WGM, int WGN, int TM, int TN, int NST>
struct Shape {
  static constexpr int BM = 32 * TM * WGM, BN = 32 * TN * WGN, NW = WGM * WGN, THREADS = 64 * NW;
  static constexpr int A_BYTES = BM * KT * 2, B_BYTES = BN * KT * 2, STAGE = A_BYTES + B_BYTES;
  static constexpr int AI = A_BYTES / 1024 / NW, BI = B_BYTES / 1024 / NW, LPT = AI + BI;
  static constexpr int PATCH = (TM < 2 ? 32 : 64) * 32 * TN * 4;      // 32 or 64 rows of a wave's sub-tile in fp32
  static constexpr int LDS = NST * STAGE > NW * PATCH ? NST * STAGE : NW * PATCH;
};

// What is done with the m-side fragments of substep kk beside multiplying them: nothing.
struct NoTap { template <int TM> __device__ __forceinline__ void operator()(int, const bf16x8 (&)[TM]) const {} };
// Sums of the m side's rows over k (a weight gradient's bias gradient, from the fragments that are there anyway): lane
// (li, hf) of row 32 j + li adds every other run of eight k, by dot products with ones (fp32 sums of exact products), of the
// substeps in `mask` (wave-uniform): the waves that share rows deal the four of a k-tile out among them.
template <int TM>
struct RowSums {
  static constexpr int CH = TM < 4 ? 2 : 1;      // chains
  float s[CH][TM];
  int mask;
  __device__ __forceinline__ void operator()(int kk, const bf16x8 (&fm)[TM]) {
    if (!(mask >> kk & 1)) return;
    const bf16x2 ones = {(bf16_t)1.f, (bf16_t)1.f};
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const bf16x2 v = {fm[j][2 * e], fm[j][2 * e + 1]};
        s[e % CH][j] = __builtin_amdgcn_fdot2_f32_bf16(v, ones, s[e % CH][j], false);
      }
  }
};

// The k-tiles [t0, t1) of the tile at (m0, n0), K the length of the whole reduction; `before_last` runs in front of the last
// k-tile's matrix instructions (all loads of operands are done by then).
template <class SH, int WGN, int TM, int TN, int NST, class LA, class LB, class F, class TAP>
__device__ __forceinline__ void multiply(const LA& A, const LB& B, int m0, int n0, int t0, int t1, int K, char* smem,
                                         f32x16 (&acc)[TN][TM], F before_last, TAP&& tap) {
  constexpr int BM = SH::BM, BN = SH::BN, AI = SH::AI, BI = SH::BI, LPT = SH::LPT, STAGE = SH::STAGE;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave / WGN) * 32 * TM, wn = (wave % WGN) * 32 * TN;
  const int li = lane & 31, hf = lane >> 5;
  const int n_row = nmap(li);
  const int c4 = lane & 3, half16 = (lane >> 4) & 1, kq = (lane & 15) >> 2;
  const int n_rowbase_t = nmap(16 * half16 + 4 * c4), m_rowbase_t = 16 * half16 + 4 * c4;
  const int nt = t1 - t0;
  const int full = K / KT - t0;            // k-tiles from t0 on that are whole

  typename LA::template State<BM, AI> sa;
  typename LB::template State<BN, BI> sb;
  A.template init<BM, AI>(sa, m0, wave * AI, lane, t0 * KT);
  B.template init<BN, BI>(sb, n0, wave * BI, lane, t0 * KT);
  auto load = [&](auto partial, int i, char* dst, int t) {
    constexpr bool P = decltype(partial)::value;
    if (i < AI) A.template issue<P, BM, AI>(sa, i, dst, wave * AI, lane, t0 + t, K);
    else B.template issue<P, BN, BI>(sb, i - AI, dst + SH::A_BYTES, wave * BI, lane, t0 + t, K);
  };
  auto issue = [&](int stage, int t) {
    char* dst = smem + stage * STAGE;
    if (t < full) {
#pragma unroll
      for (int i = 0; i < LPT; ++i) load(std::false_type{}, i, dst, t);
    } else {
#pragma unroll
      for (int i = 0; i < LPT; ++i) load(std::true_type{}, i, dst, t);
    }
  };
  // A steady k-tile's loads go out in PARTS substeps, the first of them the one behind the barrier that frees the stage: a
  // burst of loads fills the memory pipeline's queue and holds back the matrix instructions behind it.
  constexpr int PARTS = NST >= 3 ? 4 : 2;
  auto wait = [&](int younger) {           // the oldest k-tile in flight has landed; `younger` ones were issued after it
    if (NST >= 4 && younger >= 3) wait_barrier<(NST >= 4 ? 3 : 0) * LPT>();
    else if (NST >= 3 && younger >= 2) wait_barrier<(NST >= 3 ? 2 : 0) * LPT>();
    else if (younger >= 1) wait_barrier<LPT>();
    else wait_barrier<0>();
  };
  // fragment r of substep kk: n side first
  auto read1 = [&](const char* as, int kk, int r, bf16x8 (&fn)[TN], bf16x8 (&fm)[TM]) {
    const char* bs = as + SH::A_BYTES;
    if (r < TN)
      fn[r] = LB::KC ? frag_kc(bs, wn + 32 * r + n_row, 2 * kk + hf)
                     : frag_t<BN>(bs, wn + 32 * r + n_rowbase_t, 16 * kk + 8 * hf + kq);
    else
      fm[r - TN] = LA::KC ? frag_kc(as, wm + 32 * (r - TN) + li, 2 * kk + hf)
                          : frag_t<BM>(as, wm + 32 * (r - TN) + m_rowbase_t, 16 * kk + 8 * hf + kq);
  };
  // The matrix instructions of one substep, with the next substep's fragment reads between the first of them (they have to
  // land before the next substep; the compiler by itself puts them last and waits for them at once) and NL of a k-tile's
  // loads between the last.
  auto substep = [&](auto reads, bf16x8 (&fn)[TN], bf16x8 (&fm)[TM], const char* next, int kk, bf16x8 (&gn)[TN], bf16x8 (&gm)[TM], auto nload,
                     auto load_at) {
    constexpr int NMF = TM * TN, NR = TM + TN, RD = NMF >= 4 ? NMF / 2 : 1, NL = decltype(nload)::value, LD = NMF - RD + 1;
#pragma unroll
    for (int g = 0; g < NMF; ++g) {
      const int i = g / TM, j = g % TM;
      acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fn[i], fm[j], acc[i][j], 0, 0, 0);
      if (decltype(reads)::value && g < RD) {
#pragma unroll
        for (int r = g * NR / RD; r < (g + 1) * NR / RD; ++r) read1(next, kk, r, gn, gm);
      }
      __builtin_amdgcn_sched_barrier(0);
      if (g >= RD - 1) {
        const int u = g - RD + 1;
#pragma unroll
        for (int l = u * NL / LD; l < (u + 1) * NL / LD; ++l) load_at(l);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    tap((kk + 3) & 3, fm);
  };
  typedef std::integral_constant<int, 0> None;
  auto no_load = [](int) {};
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  if (nt <= 0) { before_last(); return; }

  const int pre = nt < NST ? nt : NST;
#pragma unroll 1
  for (int s = 0; s < pre; ++s) issue(s, s);
  bf16x8 fn0[TN], fm0[TM], fn1[TN], fm1[TM];
  wait(pre - 1);
#pragma unroll
  for (int r = 0; r < TM + TN; ++r) read1(smem, 0, r, fn0, fm0);
  int st = 0, t = 0;
  // substeps 0 .. 2 of the k-tile in stage st, with parts 1 .. of k-tile t - 1 + NST, which goes to stage `pend`
  auto head = [&](auto pending, int pend) {
    constexpr bool L = decltype(pending)::value;
    const char* sm = smem + st * STAGE;
    char* dst = smem + pend * STAGE;
    constexpr int P1 = L ? part_of(LPT, PARTS, 1) : 0, P2 = L && PARTS == 4 ? part_of(LPT, PARTS, 2) : 0,
                  P3 = L && PARTS == 4 ? part_of(LPT, PARTS, 3) : 0;
    substep(std::true_type{}, fn0, fm0, sm, 1, fn1, fm1, std::integral_constant<int, P1>{},
            [&](int l) { load(std::false_type{}, LPT / PARTS + l, dst, t - 1 + NST); });
    substep(std::true_type{}, fn1, fm1, sm, 2, fn0, fm0, std::integral_constant<int, P2>{},
            [&](int l) { load(std::false_type{}, 2 * LPT / PARTS + l, dst, t - 1 + NST); });
    substep(std::true_type{}, fn0, fm0, sm, 3, fn1, fm1, std::integral_constant<int, P3>{},
            [&](int l) { load(std::false_type{}, 3 * LPT / PARTS + l, dst, t - 1 + NST); });
  };
  int pend = 0;
  const int steady = nt < full ? nt : full;
  auto step = [&](auto pending) {          // the k-tile that is asked for exists and is whole
    head(pending, pend);
    wait_barrier<(NST - 2) * LPT>();       // k-tile t + 1 has landed, and every wave has read all of k-tile t
    pend = st;
    st = st + 1 == NST ? 0 : st + 1;
    substep(std::true_type{}, fn1, fm1, smem + st * STAGE, 0, fn0, fm0, std::integral_constant<int, part_of(LPT, PARTS, 0)>{},
            [&](int l) { load(std::false_type{}, l, smem + pend * STAGE, t + NST); });
    ++t;
  };
  if (NST < steady) {
    step(std::false_type{});
    while (t + NST < steady) step(std::true_type{});
#pragma unroll
    for (int i = LPT / PARTS; i < LPT; ++i) load(std::false_type{}, i, smem + pend * STAGE, t - 1 + NST);
  }
  for (; t + 1 < nt; ++t) {
    head(std::false_type{}, 0);
    const bool more = t + NST < nt;
    wait(more ? NST - 2 : nt - t - 2);
    if (more) issue(st, t + NST);
    st = st + 1 == NST ? 0 : st + 1;
    substep(std::true_type{}, fn1, fm1, smem + st * STAGE, 0, fn0, fm0, None{}, no_load);
  }
  before_last();
  __builtin_amdgcn_sched_barrier(0);
  head(std::false_type{}, 0);
  substep(std::false_type{}, fn1, fm1, nullptr, 0, fn0, fm0, None{}, no_load);
}

// The fused epilogue on 8 consecutive columns n..n+7 of row m.
__device__ __forceinline__ void epilogue8(const Epilogue& e, int m, int n, float* v) {
  if (e.bias) {
    f32x4 b0 = *reinterpret_cast<const f32x4*>(e.bias + n), b1 = *reinterpret_cast<const f32x4*>(e.bias + n + 4);
#pragma unroll
    for (int x = 0; x < 4; ++x) { v[x] += b0[x]; v[4 + x] += b1[x]; }
  }
  if (e.pre) {
    bf16x8 w;
#pragma unroll
    for (int x = 0; x < 8; ++x) w[x] = (bf16_t)v[x];
    *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16_t*>(e.pre) + (size_t)m * e.ldc + n) = w;
  }
  if (e.act == ACT_RELU) {
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] = fmaxf(v[x], 0.f);
  } else if (e.act == ACT_GELU) {
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] = gelu_f(v[x]);
  }
  if (e.dact != ACT_NONE) {
    bf16x8 s = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16_t*>(e.dact_src) + (size_t)m * e.ldd + n);
    if (e.dact == ACT_RELU) {
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] = (float)s[x] > 0.f ? v[x] : 0.f;
    } else {
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] *= dgelu_f((float)s[x]);
    }
  }
  if (e.res) {
    bf16x8 r = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16_t*>(e.res) + (size_t)m * e.ldr + n);
#pragma unroll
    for (int x = 0; x < 8; ++x) v[x] += (float)r[x];
  }
  if (e.c_f32) {
    float* cp = reinterpret_cast<float*>(e.C) + (size_t)m * e.ldc + n;
    if (e.accumulate) {
      f32x4 c0 = *reinterpret_cast<const f32x4*>(cp), c1 = *reinterpret_cast<const f32x4*>(cp + 4);
#pragma unroll
      for (int x = 0; x < 4; ++x) { v[x] += c0[x]; v[4 + x] += c1[x]; }
    }
    f32x4 o0 = {v[0], v[1], v[2], v[3]}, o1 = {v[4], v[5], v[6], v[7]};
    *reinterpret_cast<f32x4*>(cp) = o0;
    *reinterpret_cast<f32x4*>(cp + 4) = o1;
  } else {
    bf16_t* cp = reinterpret_cast<bf16_t*>(e.C) + (size_t)m * e.ldc + n;
    if (e.accumulate) {
      bf16x8 c0 = *reinterpret_cast<const bf16x8*>(cp);
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] += (float)c0[x];
    }
    bf16x8 w;
#pragma unroll
    for (int x = 0; x < 8; ++x) w[x] = (bf16_t)v[x];
    *reinterpret_cast<bf16x8*>(cp) = w;
  }
}

// Per-column sums of a wave's rows around the first row's value (lane: 8 columns, every RPI-th row; the same in all lanes of
// a column after reduce).
template <int TN>
struct ColumnSums {
  float s0[8], s1[8], p[8];
  __device__ __forceinline__ void add(const bf16x8& w, bool first, int lane) {
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const float v = (float)w[x];
      if (first) { p[x] = __shfl(v, lane % (4 * TN), 64); s0[x] = 0.f; s1[x] = 0.f; }
      const float t = v - p[x];
      s0[x] += t;
      s1[x] += t * t;
    }
  }
  __device__ __forceinline__ void reduce(int) {
#pragma unroll
    for (int o = 4 * TN; o < 64; o <<= 1)
#pragma unroll
      for (int x = 0; x < 8; ++x) { s0[x] += __shfl_xor(s0[x], o, 64); s1[x] += __shfl_xor(s1[x], o, 64); }
  }
};

// The epilogue's inputs and outputs in rows: each wave turns its sub-tile around in its own patch of the (now idle) LDS, so
// that a lane holds 8 consecutive columns and every global access of 8 lanes is one whole 128-byte line (TN = 2).  In the
// accumulators a row's 128 bytes sit in two lanes: an access would touch 32 lines and use a quarter of each.
template <int TM, int TN>
struct RowStore {
  static constexpr int LPR = 4 * TN, RPI = 64 / LPR, NIT = 32 * TM / RPI;   // lanes per row, rows per access, accesses
  static constexpr int PITCH = 128 * TN;                                    // bytes
  static __device__ __forceinline__ int slot(int row, int chunk) {          // of 16-byte chunks
    return chunk ^ (TN == 2 ? row & 15 : (row >> 1) & 7);
  }
  bf16x8 in[NIT];              // activation source or residual, asked for before the last k-tile is multiplied
  float bias[8];

  __device__ __forceinline__ void prefetch(const Epilogue& e, int mb, int nb, int M, int N, int lane) {
    const bool d = e.dact != ACT_NONE;
    const int n = nb + 8 * (lane % LPR), nc = n < N ? n : 0;
    if (d || e.res) {
      const bf16_t* src = reinterpret_cast<const bf16_t*>(d ? e.dact_src : e.res) + nc;
      const int64_t ld = d ? e.ldd : e.ldr;
#pragma unroll
      for (int I = 0; I < NIT; ++I) {
        int m = mb + I * RPI + lane / LPR;
        m = m < M ? m : M - 1;
        in[I] = *reinterpret_cast<const bf16x8*>(src + (size_t)m * ld);
      }
    }
    if (e.bias) {
      const f32x4 b0 = *reinterpret_cast<const f32x4*>(e.bias + nc), b1 = *reinterpret_cast<const f32x4*>(e.bias + nc + 4);
#pragma unroll
      for (int x = 0; x < 4; ++x) { bias[x] = b0[x]; bias[4 + x] = b1[x]; }
    }
  }
  // `raw`: partial sums, stored as fp32 at raw[m * N + n].  STATS: also the column sums of the stored bf16 values (whole tiles).
  template <bool STATS>
  __device__ __forceinline__ void store(const Epilogue& e, const f32x16 (&acc)[TN][TM], char* patch, int mb, int nb, int M,
                                        int N, int lane, float* raw, ColumnSums<TN>& cs) {
    const int li = lane & 31, hf = lane >> 5;
    const int rc = lane % LPR, n = nb + 8 * rc;
    const bool d = e.dact != ACT_NONE;
    constexpr int PJ = TM < 2 ? 1 : 2, IPJ = 32 / RPI;       // 32-row pieces in the patch, accesses per piece
#pragma unroll
    for (int I = 0; I < NIT; ++I) {
      if (I % (IPJ * PJ) == 0) {
#pragma unroll
        for (int jj = 0; jj < PJ; ++jj) {
          const int j = I / IPJ + jj, row = 32 * jj + li;
          if (j >= TM) break;
#pragma unroll
          for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const f32x4 o = {acc[i][j][4 * c], acc[i][j][4 * c + 1], acc[i][j][4 * c + 2], acc[i][j][4 * c + 3]};
              *reinterpret_cast<f32x4*>(patch + row * PITCH + 16 * slot(row, 8 * i + 4 * (c >> 1) + 2 * hf + (c & 1))) = o;
            }
        }
      }
      const int row = (I % (IPJ * PJ)) * RPI + lane / LPR, m = mb + I * RPI + lane / LPR;
      const f32x4 a = *reinterpret_cast<const f32x4*>(patch + row * PITCH + 16 * slot(row, 2 * rc));
      const f32x4 b = *reinterpret_cast<const f32x4*>(patch + row * PITCH + 16 * slot(row, 2 * rc + 1));
      if (!STATS && (m >= M || n >= N)) continue;
      if (!STATS && raw) {
        float* p = raw + (size_t)m * N + n;
        *reinterpret_cast<f32x4*>(p) = a;
        *reinterpret_cast<f32x4*>(p + 4) = b;
        continue;
      }
      float v[8] = {a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]};
      if (e.bias) {
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] += bias[x];
      }
      if (e.pre) {
        bf16x8 w;
#pragma unroll
        for (int x = 0; x < 8; ++x) w[x] = (bf16_t)v[x];
        *reinterpret_cast<bf16x8*>(reinterpret_cast<bf16_t*>(e.pre) + (size_t)m * e.ldc + n) = w;
      }
      if (e.act == ACT_RELU) {
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = fmaxf(v[x], 0.f);
      } else if (e.act == ACT_GELU) {
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = gelu_f(v[x]);
      }
      if (d) {
        if (e.dact == ACT_RELU) {
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] = (float)in[I][x] > 0.f ? v[x] : 0.f;
        } else {
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] *= dgelu_f((float)in[I][x]);
        }
      }
      if (e.res) {
        bf16x8 r = in[I];
        if (d) r = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const bf16_t*>(e.res) + (size_t)m * e.ldr + n);
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] += (float)r[x];
      }
      if (e.c_f32) {
        float* cp = reinterpret_cast<float*>(e.C) + (size_t)m * e.ldc + n;
        f32x4 o0 = {v[0], v[1], v[2], v[3]}, o1 = {v[4], v[5], v[6], v[7]};
        if (e.accumulate) { o0 += *reinterpret_cast<const f32x4*>(cp); o1 += *reinterpret_cast<const f32x4*>(cp + 4); }
        *reinterpret_cast<f32x4*>(cp) = o0;
        *reinterpret_cast<f32x4*>(cp + 4) = o1;
      } else {
        bf16_t* cp = reinterpret_cast<bf16_t*>(e.C) + (size_t)m * e.ldc + n;
        if (e.accumulate) {
          const bf16x8 c0 = *reinterpret_cast<const bf16x8*>(cp);
#pragma unroll
          for (int x = 0; x < 8; ++x) v[x] += (float)c0[x];
        }
        bf16x8 w;
#pragma unroll
        for (int x = 0; x < 8; ++x) w[x] = (bf16_t)v[x];
        *reinterpret_cast<bf16x8*>(cp) = w;
        if (STATS) cs.add(w, I == 0, lane);
      }
    }
  }
};

// Sums `pieces` partial sums of 8 columns in order, eight loads in flight, and hands them to f.
template <class F>
__device__ __forceinline__ void add_pieces(const float* src, size_t slab, int pieces, F f) {
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  int s = 0;
  for (; s + 4 <= pieces; s += 4) {
    f32x4 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      a[u] = *reinterpret_cast<const f32x4*>(src + (s + u) * slab);
      b[u] = *reinterpret_cast<const f32x4*>(src + (s + u) * slab + 4);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int x = 0; x < 4; ++x) { v[x] += a[u][x]; v[4 + x] += b[u][x]; }
  }
  for (; s < pieces; ++s) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(src + s * slab), b = *reinterpret_cast<const f32x4*>(src + s * slab + 4);
#pragma unroll
    for (int x = 0; x < 4; ++x) { v[x] += a[x]; v[4 + x] += b[x]; }
  }
  f(v);
}

// Tile number -> coordinates: column-major groups of 8 tile rows, so that blocks that run together share operands.
__device__ __forceinline__ void tile_coords(int q, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int width = 8 * tiles_n, gid = q / width, first = gid * 8;
  const int gs = tiles_m - first < 8 ? tiles_m - first : 8, r = q - gid * width;
  tn = r / gs;
  tm = first + r - tn * gs;
}
// Work number of a block: blocks are dealt to the eight XCDs in turn; each XCD takes one contiguous range of the numbers.
__device__ __forceinline__ int xcd_range(int bid, int total) {
  const int per = total >> 3;
  return bid < per * 8 ? (bid & 7) * per + (bid >> 3) : bid;
}

}  // namespace tile

// The cheapest of the shapes in `mask` (bits: rows of the shape table) and cut for n products of one reduction length.
TilePlan tile_plan(const OpCtx& c, int n, const int* M, const int* N, int K, unsigned mask, int max_pieces);

}  // namespace lp
