// 3x3 / 1x1 convolutions over NHWC bf16 activations as implicit GEMMs on the matrix cores (gemm_tile.h).  No im2col
// buffer exists: the operand loaders gather pixels directly, 16 bytes = 8 consecutive channels per lane and load, and take
// zero padding, stride holes and what lies past the reduction's end from a zero page.
//   forward : out[(n,p,q), o]  = sum_{(r,s,c)} x[n, p*st+r-pad, q*st+s-pad, c] * w[o, r, s, c]
//   dgrad   : dx[(n,h,w), c]   = sum_{(r,s,o)} dout[n, (h+pad-r)/st, (w+pad-s)/st, o] * w[o, r, s, c]
//   wgrad   : dw[o, (r,s,c)]   = sum_{(n,p,q)} dout[(n,p,q), o] * x[n, p*st+r-pad, q*st+s-pad, c]   (fp32, cut along k)
// Needs C % 8 == 0 and O % 8 == 0; the stem convolution on 1 to 3 channels has kernels of its own (kernels_conv_stem.hip).
#include <stdio.h>
#include <type_traits>
#include "gemm_tile.h"

namespace lp {

using namespace tile;

namespace {

// k -> (k / d, k % d) by multiplication: exact for k d < 2^32 (a filter's reduction: at most 2^16 taps and channels).
struct Divider {
  unsigned m; int d;
  __host__ explicit Divider(int d_) : m((unsigned)((0xffffffffull + d_) / d_)), d(d_) {}
  __device__ __forceinline__ int quot(int k) const { return d == 1 ? k : (int)__umulhi((unsigned)k, m); }
};

// Pixel number -> (n, h, w) for numbers that start at a wave-uniform one: one division by the image size, and multiplications
// for what is added to it (a division per lane, row and filter tap made a block's start 2 to 3 us long).
struct PixelWalk {
  int w0, h0, n0, W, H;
  Divider by_w, by_h;
  __device__ __forceinline__ PixelWalk(int first, int W_, int H_, const Divider& bw, const Divider& bh)
      : W(W_), H(H_), by_w(bw), by_h(bh) {
    const int t = first / W;
    w0 = first - t * W;
    n0 = t / H;
    h0 = t - n0 * H;
  }
  __device__ __forceinline__ void at(int more, int& n, int& h, int& w) const {      // more < 2^12
    const int a = w0 + more, t = by_w.quot(a), b = h0 + t, u = by_h.quot(b);
    w = a - t * W;
    h = b - u * H;
    n = n0 + u;
  }
};

__device__ __forceinline__ const bf16_t* zero_page() { return reinterpret_cast<const bf16_t*>(kZeroPage); }

// The gathered operand of the forward pass (rows = output pixels, k = (r,s,c)) and of the data gradient (rows = input pixels,
// k = (r,s,o)).  A row's base pointer and, per filter row and column, whether the tap exists for it are worked out once; a
// tap's offset from the base is the same for all rows (data gradient: pixel (h + pad - r) / st is (h + pad) / st - r / st where
// the division leaves no remainder).  UNI: the reduction's channels are a multiple of 64, so a k-tile is one tap and its
// offset and mask bits are scalars; with the general form's per-lane arithmetic the 64-channel forward convolution of 256
// images of 32 x 32 was bound by the vector ALU (73 us).
template <bool UNI>
struct ConvGather {
  static constexpr bool KC = true;
  const bf16_t* x;
  int rows, rw, rh;          // rows; the row pixels' width and height
  int gw, gh, ch;            // the gathered image's width, height and channels
  int st, pad, R, S;         // dir > 0: gathered pixel = st * pixel + tap - pad; dir < 0: (pixel + pad - tap) / st
  int dir;
  Divider by_ch, by_s, by_st, by_rw, by_rh;
  template <int ROWS, int NI> struct State { const bf16_t* g[NI]; unsigned ok[NI]; };       // ok: bits r, and 16 + s
  template <int ROWS, int NI>
  __device__ __forceinline__ void init(State<ROWS, NI>& s, int r0, int q0, int lane, int) const {
    const PixelWalk walk(r0 + 8 * q0, rw, rh, by_rw, by_rh);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int trow, kc;
      chunk_of<true, ROWS>(q0 + i, lane, trow, kc);
      const int row = r0 + trow;
      unsigned ok = 0;
      int h0 = 0, w0 = 0, n = 0;
      if (row < rows) {
        int h, w;
        walk.at(trow - 8 * q0, n, h, w);
        if (dir > 0) {
          h0 = h * st - pad; w0 = w * st - pad;
          for (int r = 0; r < R; ++r) ok |= (unsigned)((unsigned)(h0 + r) < (unsigned)gh) << r;
          for (int c = 0; c < S; ++c) ok |= (unsigned)((unsigned)(w0 + c) < (unsigned)gw) << (16 + c);
        } else {
          h0 = by_st.quot(h + pad); w0 = by_st.quot(w + pad);
          for (int r = 0; r < R; ++r) {
            const int a = h + pad - r, q = by_st.quot(a);
            ok |= (unsigned)(a >= 0 && q * st == a && q < gh) << r;
          }
          for (int c = 0; c < S; ++c) {
            const int a = w + pad - c, q = by_st.quot(a);
            ok |= (unsigned)(a >= 0 && q * st == a && q < gw) << (16 + c);
          }
        }
      }
      s.ok[i] = ok;
      s.g[i] = x + ((int64_t)(n * gh + h0) * gw + w0) * ch + (UNI ? kc : 0);
    }
  }
  template <bool PARTIAL, int ROWS, int NI>
  __device__ __forceinline__ void issue(State<ROWS, NI>& s, int i, char* dst, int q0, int lane, int kt, int K) const {
    int k = kt * KT;
    if (!UNI) {
      int row, kc;
      chunk_of<true, ROWS>(q0 + i, lane, row, kc);
      k += kc;
    }
    const int rs = by_ch.quot(k), r = by_s.quot(rs), c = rs - r * S;
    const int tap = dir > 0 ? r * gw + c : -(by_st.quot(r) * gw + by_st.quot(c));
    const unsigned m = s.ok[i];
    bool ok = ((m >> r) & (m >> (16 + c)) & 1u) != 0;
    if (PARTIAL && !UNI) ok = ok && k < K;
    const bf16_t* src = s.g[i] + (tap * ch + (k - rs * ch));
    to_lds(ok ? src : zero_page(), dst + (q0 + i) * 1024);
  }
};

// dgrad B operand: rows = input channel c (contiguous in memory), k = (r,s,o): w[o, r, s, c].  UNI: as above.
template <bool UNI>
struct ConvFilterT {
  static constexpr bool KC = false;
  const bf16_t* w; int C, O, RS; Divider by_o;
  template <int ROWS, int NI> struct State { const bf16_t* g[NI]; };
  template <int ROWS, int NI>
  __device__ __forceinline__ void init(State<ROWS, NI>& s, int r0, int q0, int lane, int) const {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int row, k;
      chunk_of<false, ROWS>(q0 + i, lane, row, k);
      row += r0;
      s.g[i] = w + (row + 8 <= C ? row : C - 8) + (UNI ? (size_t)k * RS * C : 0);
    }
  }
  template <bool PARTIAL, int ROWS, int NI>
  __device__ __forceinline__ void issue(State<ROWS, NI>& s, int i, char* dst, int q0, int lane, int kt, int K) const {
    int k = kt * KT;
    if (!UNI) {
      int row, kr;
      chunk_of<false, ROWS>(q0 + i, lane, row, kr);
      k += kr;
    }
    const int rs = by_o.quot(k), o = k - rs * O;
    const bf16_t* src = s.g[i] + ((int64_t)o * RS + rs) * C;
    to_lds(UNI || !PARTIAL || k < K ? src : zero_page(), dst + (q0 + i) * 1024);
  }
};

// wgrad B operand: rows j = (r,s,c) (c contiguous), k = output pixel (n,p,q): gathered input patches.  A lane's pixel moves
// by 64 from k-tile to k-tile: (dn, dp, dq) with carries.  SAME (stride 1, output as large as the input): so does its address.
template <bool SAME>
struct ConvPatchT {
  static constexpr bool KC = false;
  const bf16_t* x; ConvArgs a; int J, dn, dp, dq; Divider by_c, by_s, by_q, by_p;
  template <int ROWS, int NI> struct State { const bf16_t* g[NI]; int rs[NI], n[SAME ? 1 : NI], p[NI], q[NI]; };
  template <int ROWS, int NI>
  __device__ __forceinline__ void init(State<ROWS, NI>& s, int r0, int q0, int lane, int k0) const {
    const PixelWalk walk(k0, a.Q, a.P, by_q, by_p);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      int row, k;
      chunk_of<false, ROWS>(q0 + i, lane, row, k);
      const int j = r0 + row;
      int c0 = 0, rr = 0, ss = 0;
      if (j < J) {
        const int rs = by_c.quot(j), r = by_s.quot(rs);
        rr = r - a.pad; ss = rs - r * a.S - a.pad;
        c0 = j - rs * a.C;
        s.rs[i] = rr * 65536 + ss;             // two signed halves
      } else {
        s.rs[i] = -(1 << 30);                  // above every image
      }
      int n;
      walk.at(k, n, s.p[i], s.q[i]);
      if (SAME) s.g[i] = x + ((int64_t)k0 + k + rr * a.W + ss) * a.C + c0;
      else { s.g[i] = x + c0; s.n[i] = n; }
    }
  }
  template <bool PARTIAL, int ROWS, int NI>
  __device__ __forceinline__ void issue(State<ROWS, NI>& s, int i, char* dst, int q0, int lane, int kt, int K) const {
    bool ok = true;
    if (PARTIAL) {
      int row, k;
      chunk_of<false, ROWS>(q0 + i, lane, row, k);
      ok = kt * KT + k < K;
    }
    const int sx = (short)s.rs[i], rx = (s.rs[i] - sx) >> 16;
    const int h = (SAME ? s.p[i] : s.p[i] * a.stride) + rx, w = (SAME ? s.q[i] : s.q[i] * a.stride) + sx;
    ok = ok && (unsigned)h < (unsigned)a.H && (unsigned)w < (unsigned)a.W;
    const bf16_t* src = s.g[i];
    if (!SAME) src += (int64_t)((s.n[i] * a.H + h) * a.W + w) * a.C;
    to_lds(ok ? src : zero_page(), dst + (q0 + i) * 1024);
    if (SAME) s.g[i] += KT * a.C;
    int q = s.q[i] + dq, p = s.p[i] + dp;
    if (q >= a.Q) { q -= a.Q; ++p; }
    const bool wrap = p >= a.P;
    if (wrap) p -= a.P;
    if (!SAME) s.n[i] += dn + (wrap ? 1 : 0);
    s.q[i] = q; s.p[i] = p;
  }
};

template <class L> struct IsForward { static constexpr bool value = false; };
template <bool UNI> struct Forward : ConvGather<UNI> {
  explicit Forward(const ConvGather<UNI>& g) : ConvGather<UNI>(g) {}
};
template <bool UNI> struct IsForward<Forward<UNI>> { static constexpr bool value = true; };

// One output tile.  STATS (the convolution in front of a batch normalisation; one piece, whole tiles): the block also leaves,
// per output column, the sums the normalisation needs over the rows of the tile, taken from the rounded values it stores:
// p = the tile's first row, s0 = sum (z - p), s1 = sum (z - p)^2, in ws as [3][M / BM][N] (s0, s1, p).
template <class LA, class LB, int WGM, int WGN, int TM, int TN, int NST, bool STATS>
__global__ void __launch_bounds__(64 * WGM * WGN, WGM * WGN == 8 || (Shape<WGM, WGN, TM, TN, NST>::LDS <= 80 * 1024) ? 2 : 1)
k_conv_tile(LA A, LB B, Epilogue e, int M, int N, int K, int tiles_m, int tiles_n, int splits, int per, float* ws) {
  typedef Shape<WGM, WGN, TM, TN, NST> SH;
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int w = xcd_range(blockIdx.x, gridDim.x);
  const int tiles = tiles_m * tiles_n, piece = w / tiles;
  w -= piece * tiles;
  int tm, tn;
  tile_coords(w, tiles_m, tiles_n, tm, tn);
  const int nt = (K + KT - 1) / KT, t0 = piece * per, t1 = t0 + per < nt ? t0 + per : nt;
  const int mb = tm * SH::BM + (wave / WGN) * 32 * TM, nb = tn * SH::BN + (wave % WGN) * 32 * TN;
  const bool raw = splits > 1;
  f32x16 acc[TN][TM];
  RowStore<TM, TN> out;
  multiply<SH, WGN, TM, TN, NST>(A, B, tm * SH::BM, tn * SH::BN, t0, t1, K, smem, acc,
                                 [&] { if (!raw) out.prefetch(e, mb, nb, M, N, lane); }, NoTap{});
  __syncthreads();
  ColumnSums<TN> cs;
  out.template store<STATS>(e, acc, smem + wave * SH::PATCH, mb, nb, M, N, lane, raw ? ws + (size_t)piece * M * N : nullptr, cs);
  if constexpr (STATS) {
    // The waves that share columns leave their sums in LDS, and the first of them shifts the others to its pivot
    // (d = p_w - p: s0 += s0_w + n d, s1 += s1_w + 2 d s0_w + n d^2) in wave order.
    __syncthreads();
    float* sh = reinterpret_cast<float*>(smem);               // [waves][3][32 TN]
    cs.reduce(lane);
    if (lane < 4 * TN) {
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        sh[(wave * 3 + 0) * 32 * TN + 8 * lane + x] = cs.s0[x];
        sh[(wave * 3 + 1) * 32 * TN + 8 * lane + x] = cs.s1[x];
        sh[(wave * 3 + 2) * 32 * TN + 8 * lane + x] = cs.p[x];
      }
    }
    __syncthreads();
    if (wave < WGN && lane < 32 * TN) {
      const float* mine = sh + wave * 3 * 32 * TN + lane;
      float s0 = mine[0], s1 = mine[32 * TN];
      const float p = mine[64 * TN], n = 32.f * TM;
#pragma unroll
      for (int u = 1; u < WGM; ++u) {
        const float* o = sh + (u * WGN + wave) * 3 * 32 * TN + lane;
        const float o0 = o[0], d = o[64 * TN] - p;
        s0 += o0 + n * d;
        s1 += o[32 * TN] + 2.f * d * o0 + n * d * d;
      }
      const size_t nslab = (size_t)M / SH::BM, slab = tm;
      float* sp = ws + slab * N + nb + lane;
      sp[0] = s0;
      sp[nslab * N] = s1;
      sp[2 * nslab * N] = p;
    }
  }
}

// Adds the pieces' partial sums in a fixed order and applies the epilogue; LANES lanes share 8 consecutive columns (lane u
// takes pieces u, u + LANES, ..., the lanes' sums are then added as a tree), so that a small filter gradient in many pieces
// is not one thread's chain of loads (24 x 216 in 62 pieces: 7.5 us with one lane).
template <int LANES>
__device__ __forceinline__ void reduce_block(const float* ws, const Epilogue& e, int M, int N, int splits, int block) {
  const size_t idx = ((size_t)block * 256 + threadIdx.x) / LANES;
  const int u = threadIdx.x % LANES, n8 = N >> 3;
  const bool in = idx < (size_t)M * n8;
  const int m = in ? (int)(idx / n8) : 0, n = in ? (int)(idx % n8) * 8 : 0;
  const size_t slab = (size_t)M * N;
  add_pieces(ws + (size_t)m * N + n + u * slab, LANES * slab, (splits - u + LANES - 1) / LANES, [&](float* v) {
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1)
#pragma unroll
      for (int x = 0; x < 8; ++x) v[x] += __shfl_xor(v[x], o, 64);
    if (in && u == 0) epilogue8(e, m, n, v);
  });
}
template <int LANES>
__global__ void __launch_bounds__(256) k_conv_reduce(const float* __restrict__ ws, Epilogue e, int M, int N, int splits) {
  reduce_block<LANES>(ws, e, M, N, splits, blockIdx.x);
}
int reduce_lanes(int M, int N, int splits) { return (size_t)M * (N / 8) < 16384 && splits >= 8 ? 8 : 1; }
unsigned reduce_blocks(int M, int N, int lanes) { return (unsigned)(((size_t)M * (N / 8) * lanes + 255) / 256); }

// The same for the filter gradients of a stage's backward pass, each in its own blocks (first[i]: the first of gradient i's).
// Alone each is a few KB to a few MB of sums, bound by a launch and two memory latencies (5 us) in the middle of the chain of a
// backward pass; together they cost one such launch a stage, with the same bits.  A step, before and after in turn on one card: four
// stages of batch 256 (64 channels) 2620 and 2598 us (runs of one side 0.1 % apart), with batch 128 and one head 2308 and 2257; of
// three stages of 24 channels on 28 x 28 it is lost in the noise of the host's issue (6 to 10 %).
struct FilterTable { PendingFilters::Filter f[kMaxFilters]; int lanes[kMaxFilters], first[kMaxFilters]; int count; };
__global__ void __launch_bounds__(256) k_conv_reduce_filters(FilterTable t) {
  int p = 0;
#pragma unroll
  for (int i = 1; i < kMaxFilters; ++i)
    if (i < t.count && (int)blockIdx.x >= t.first[i]) p = i;
  Epilogue e = {};
  e.C = t.f[p].dw; e.ldc = t.f[p].N; e.c_f32 = 1; e.accumulate = t.f[p].accumulate;
  const int block = blockIdx.x - t.first[p];
  if (t.lanes[p] == 8) reduce_block<8>(t.f[p].ws, e, t.f[p].M, t.f[p].N, t.f[p].splits, block);
  else reduce_block<1>(t.f[p].ws, e, t.f[p].M, t.f[p].N, t.f[p].splits, block);
}

// `loaders` names the two loader types as a profiler prints them: the launch is timed under the kernel's name.  pieces: where the
// sums of a product in several pieces go.  st (forward
// convolutions only): if the launch qualifies (whole tiles, one piece, room in st->buf) the kernel also leaves the
// normalisation's column statistics per tile there, and st->nslab / st->slab_rows say how many.
template <class LA, class LB, int WGM, int WGN, int TM, int TN, int NST>
hipError_t launch_shape(const OpCtx& c, const LA& A, const LB& B, const Epilogue& e, int M, int N, int K, const TilePlan& plan,
                        const char* loaders, ConvStats* st, float* pieces) {
  typedef Shape<WGM, WGN, TM, TN, NST> SH;
  const int tm = (M + SH::BM - 1) / SH::BM, tn = (N + SH::BN - 1) / SH::BN;
  bool stats = false;
  if constexpr (IsForward<LA>::value) {
    if (st && st->buf && plan.splits == 1 && M % SH::BM == 0 && N % SH::BN == 0 && (size_t)3 * tm * N <= st->cap) {
      stats = true; st->nslab = tm; st->slab_rows = SH::BM;
    }
  }
  static char names[2][112];
  char* name = names[stats];
  if (!name[0])
    snprintf(name, sizeof names[0], "k_conv_tile<%s, %d, %d, %d, %d, %d, %s>", loaders, WGM, WGN, TM, TN, NST, stats ? "true" : "false");
  ProfScope one_(c, KC_GEMM_KERNEL, 2.0 * M * N * K, 0, name);
  auto go = [&](auto flag, float* ws) -> hipError_t {
    constexpr bool STATS = decltype(flag)::value;
    auto fn = k_conv_tile<LA, LB, WGM, WGN, TM, TN, NST, STATS>;
    if (SH::LDS > 64 * 1024) {
      static LdsLimit limit;
      hipError_t err = limit.raise(reinterpret_cast<const void*>(fn), SH::LDS);
      if (err != hipSuccess) return err;
    }
    fn<<<tm * tn * plan.splits, SH::THREADS, SH::LDS, c.stream>>>(A, B, e, M, N, K, tm, tn, plan.splits, plan.per, ws);
    return hipGetLastError();
  };
  if constexpr (IsForward<LA>::value) {
    if (stats) return go(std::true_type{}, st->buf);
  }
  return go(std::false_type{}, pieces);
}

// Tile shapes beside those of the dense products: 256 x 64 and 64 x 128 for 64-channel convolutions and their filter gradients;
// 128 x 32 where the output has at most 32 columns (65536 pixels x 16 channels: 12.0 us with 64 columns, 8.8 with 32; with
// more columns than that it loses to 64 x 64: 2450 x 96 16.9 against 9.9 us).
TilePlan conv_plan(const OpCtx& c, int M, int N, int K) {
  const unsigned mask = 0x1f | 1u << 6 | 1u << 7 | (N <= 32 ? 1u << 8 : 0u);
  return tile_plan(c, 1, &M, &N, K, mask, 64);
}
// later: the product is a filter gradient that may leave its pieces in c.filters.
template <class LA, class LB>
hipError_t conv_product(const OpCtx& c, const LA& A, const LB& B, const Epilogue& e, int M, int N, int K, const char* loaders,
                        ConvStats* st = nullptr, float* later = nullptr, int accumulate = 0) {
  const TilePlan plan = conv_plan(c, M, N, K);
  const size_t need = plan.splits > 1 ? (size_t)plan.splits * M * N : 0;
  if (need && c.filters && (c.filters->used + need > c.splitk_elems || c.filters->count == kMaxFilters)) {
    hipError_t e0 = op_conv_add_pending(c);
    if (e0 != hipSuccess) return e0;
  }
  float* ws = need && c.filters ? c.splitk_ws + c.filters->used : c.splitk_ws;
  hipError_t err = hipErrorInvalidValue;
  switch (plan.shape) {
    case 0: err = launch_shape<LA, LB, 2, 2, 1, 1, 4>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 1: err = launch_shape<LA, LB, 2, 2, 2, 1, 3>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 2: err = launch_shape<LA, LB, 2, 2, 2, 2, 2>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 3: err = launch_shape<LA, LB, 2, 2, 2, 2, 4>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 4: err = launch_shape<LA, LB, 4, 2, 2, 2, 3>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 6: err = launch_shape<LA, LB, 2, 2, 1, 2, 3>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 7: err = launch_shape<LA, LB, 4, 1, 2, 2, 2>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
    case 8: err = launch_shape<LA, LB, 4, 1, 1, 1, 2>(c, A, B, e, M, N, K, plan, loaders, st, ws); break;
  }
  if (err != hipSuccess || plan.splits == 1) return err;
  if (later && c.filters) {
    c.filters->f[c.filters->count++] = PendingFilters::Filter{ws, later, M, N, plan.splits, accumulate};
    c.filters->used += need;
    return hipSuccess;
  }
  const int lanes = reduce_lanes(M, N, plan.splits);
  if (lanes == 8) k_conv_reduce<8><<<reduce_blocks(M, N, 8), 256, 0, c.stream>>>(ws, e, M, N, plan.splits);
  else k_conv_reduce<1><<<reduce_blocks(M, N, 1), 256, 0, c.stream>>>(ws, e, M, N, plan.splits);
  return hipGetLastError();
}

Epilogue plain_epilogue(void* C, int64_t ldc, int c_f32, int accumulate) {
  GemmArgs g; g.C = C; g.ldc = ldc; g.c_f32 = c_f32; g.accumulate = accumulate;
  return make_epilogue(g);
}

bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// Beside the alignment: a filter's rows and columns are bits of 16, pixel coordinates travel in 16 bits, and a Divider's products stay
// below 2^32.
bool conv_mfma_ok(const OpCtx& c, const ConvArgs& a, const void* p0, const void* p1, const void* p2) {
  const int64_t ch = a.C > a.O ? a.C : a.O;
  const bool small = a.H + 2 * a.pad < (1 << 14) && a.W + 2 * a.pad < (1 << 14) && a.R <= 16 && a.S <= 16 && a.R * a.S * ch * ch < ((int64_t)1 << 31);
  return c.dt == BF16 && a.C % 8 == 0 && a.O % 8 == 0 && a.C >= 8 && a.O >= 8 && small && al16(p0) && al16(p1) && al16(p2);
}

// The tiles that a convolution's forward (0), data-gradient (1) or filter-gradient (2) product takes.
TilePlan conv_mfma_plan(const OpCtx& c, const ConvArgs& a, int dir) {
  const int pixels = a.N * a.P * a.Q, taps = a.R * a.S;
  if (dir == 0) return conv_plan(c, pixels, a.O, taps * a.C);
  if (dir == 1) return conv_plan(c, a.N * a.H * a.W, a.C, taps * a.O);
  return conv_plan(c, a.O, taps * a.C, pixels);
}
hipError_t conv_fwd_mfma(const OpCtx& c, const ConvArgs& a, const void* x, const void* w, void* out, ConvStats* st) {
  const int M = a.N * a.P * a.Q, K = a.R * a.S * a.C;
  if (M <= 0) return hipSuccess;
  const DenseLoader<true> B{Operand{(const bf16_t*)w, K, a.O}};
  const Epilogue e = plain_epilogue(out, a.O, 0, 0);
  auto go = [&](auto uni, const char* name) {
    constexpr bool U = decltype(uni)::value;
    const Forward<U> A(ConvGather<U>{(const bf16_t*)x, M, a.Q, a.P, a.W, a.H, a.C, a.stride, a.pad, a.R, a.S, 1, Divider(a.C),
                                     Divider(a.S), Divider(1), Divider(a.Q), Divider(a.P)});
    return conv_product(c, A, B, e, M, a.O, K, name, st);
  };
  return a.C % KT == 0 ? go(std::true_type{}, "Forward<true>, tile::DenseLoader<true>")
                       : go(std::false_type{}, "Forward<false>, tile::DenseLoader<true>");
}
hipError_t conv_bwd_data_mfma(const OpCtx& c, const ConvArgs& a, const void* dout, const void* w, void* dx,
                              const void* add) {
  const int M = a.N * a.H * a.W, K = a.R * a.S * a.O;
  if (M <= 0) return hipSuccess;
  Epilogue e = plain_epilogue(dx, a.C, 0, 0);
  e.res = add; e.ldr = a.C;      // a tensor of the output's shape added to the result
  auto go = [&](auto uni, const char* name) {
    constexpr bool U = decltype(uni)::value;
    const ConvGather<U> A{(const bf16_t*)dout, M, a.W, a.H, a.Q, a.P, a.O, a.stride, a.pad, a.R, a.S, -1, Divider(a.O),
                          Divider(a.S), Divider(a.stride), Divider(a.W), Divider(a.H)};
    const ConvFilterT<U> B{(const bf16_t*)w, a.C, a.O, a.R * a.S, Divider(a.O)};
    return conv_product(c, A, B, e, M, a.C, K, name);
  };
  return a.O % KT == 0 ? go(std::true_type{}, "ConvGather<true>, ConvFilterT<true>")
                       : go(std::false_type{}, "ConvGather<false>, ConvFilterT<false>");
}
hipError_t conv_bwd_weight_mfma(const OpCtx& c, const ConvArgs& conv, const void* dout, const void* x, float* dw,
                                int accumulate) {
  ConvArgs a = conv;
  const int K = a.N * a.P * a.Q, J = a.R * a.S * a.C;
  if (K <= 0) a.P = a.Q = 1;      // no output pixels (a filter larger than the image): a sum of none, with divisors above zero
  const DenseLoader<false> A{Operand{(const bf16_t*)dout, a.O, a.O}};
  const Epilogue e = plain_epilogue(dw, J, 1, accumulate);
  auto go = [&](auto same, const char* name) {
    constexpr bool S = decltype(same)::value;
    const ConvPatchT<S> B{(const bf16_t*)x, a, J, KT / (a.P * a.Q), KT / a.Q % a.P, KT % a.Q, Divider(a.C), Divider(a.S), Divider(a.Q), Divider(a.P)};
    return conv_product(c, A, B, e, a.O, J, K, name, nullptr, dw, accumulate);
  };
  return a.stride == 1 && a.P == a.H && a.Q == a.W ? go(std::true_type{}, "tile::DenseLoader<false>, ConvPatchT<true>")
                                                   : go(std::false_type{}, "tile::DenseLoader<false>, ConvPatchT<false>");
}


hipError_t op_conv_add_pending(const OpCtx& c) {
  PendingFilters* ps = c.filters;
  if (!ps || ps->count == 0) return hipSuccess;
  FilterTable t = {};
  int blocks = 0;
  for (int i = 0; i < ps->count; ++i) {
    const PendingFilters::Filter& f = t.f[i] = ps->f[i];
    t.lanes[i] = reduce_lanes(f.M, f.N, f.splits);
    t.first[i] = blocks;
    blocks += (int)reduce_blocks(f.M, f.N, t.lanes[i]);
  }
  t.count = ps->count;
  ps->count = 0; ps->used = 0;
  k_conv_reduce_filters<<<blocks, 256, 0, c.stream>>>(t);
  return hipGetLastError();
}

}  // namespace lp
