// Causal multi-head attention on the CDNA4 matrix cores (bf16 operands, fp32 accumulation and
// softmax), head sizes 16, 32 and 64, flash-style: the S x S score matrix lives only in registers.
// (64 sequences of 128, 8 heads of 16, on the plain kernels: forward 112 us, backward 149 + 287 us.  Here 7.9 us and
// 22.8 us for both backward kernels.  The head size only changes the number of 16-deep products of a
// score tile and of 32-row output tiles; a 16-wide head leaves half of its one output tile unused, which costs
// nothing that counts, since the exponentials bound the kernels.)
//
// All three kernels keep the score tile transposed where that puts one query per lane column, so
// that the running max / sum / log-sum-exp of a query are lane-uniform scalars:
//   forward : S^T[key, q] = K Q^T  -> online softmax ->  O^T[dh, q] += V^T P^T
//   dQ      : S^T, dP^T[key, q] = V dO^T -> dS^T -> dQ^T[dh, q] += K^T dS^T
//   dK, dV  : S[q, key] = Q K^T, dP[q, key] = dO V^T -> P, dS -> dV^T[dh, key] += dO^T P,
//             dK^T[dh, key] += Q^T dS
// P and dS of heads of 64 are rounded to bf16 for the second products; those of narrower heads stay in fp32 (split8).
// Three matrix instructions instead of one there, measured over the rounded form: 64 sequences of 128, 8 heads of 16,
// forward 7.1 -> 7.9 us, backward 18.7 -> 22.8 us; 4 of 2048, 8 heads of 32, 29.2 -> 46.2 us and 77 -> 122 us (backward: both launches).
// The accumulator layout of v_mfma_f32_32x32x16_bf16 (value v of lane l: row 8*(v/4) + 4*(l/32) + v%4,
// column l%32) is exactly the B-operand layout of the next MFMA over the row index, so P and dS
// never pass through LDS.  Operands whose reduction index is the slow one in memory (V for the
// forward, K for dQ, Q and dO for dK/dV) sit in LDS as in memory and are read with the transposing LDS
// read (ds_read_b64_tr_b16).  The next tile's global loads are issued before the current tile's MFMAs.
// Layout: qkv [B*S, 3*H*DH] (q | k | v, head h at columns h*DH..), o [B*S, H*DH], lse [B, H, S].
#include "common.h"
#include "gemm_common.h"

namespace lp {

// Padded LDS row: the head size + 8 elements (144 or 80 bytes); a 16-wide head takes the 32-wide row, because the
// transposing reads cover 32 columns (what they find past the head lands in output rows that are not written).
template <int DH> constexpr int kAld = DH == 64 ? 72 : 40;
template <int DH> constexpr float kScale = DH == 64 ? 0.125f : (DH == 32 ? 0.17677669529663687f : 0.25f);
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#define MFMA32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16((a), (b), (c), 0, 0, 0)

__device__ __forceinline__ bf16x8 zero8() {
  bf16x8 z;
#pragma unroll
  for (int i = 0; i < 8; ++i) z[i] = (bf16_t)0.f;
  return z;
}
__device__ __forceinline__ void zero16(f32x16& a) {
#pragma unroll
  for (int i = 0; i < 16; ++i) a[i] = 0.f;
}
// 8 accumulator values -> bf16 B-operand fragment (values 8*kk .. 8*kk+7 of a 32x32 tile)
__device__ __forceinline__ bf16x8 pack8(const f32x16& a, int kk) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16_t)a[8 * kk + e];
  return r;
}
// B-operand fragments of the same eight values.  Heads of 64 take one, rounded to bf16.  Narrower heads keep P and dS in
// fp32: the three fragments are the value's top, middle and last eight bits (cut, not rounded), whose sum is the value, and
// their products with the bf16 operand are exact, so that the sums are fp32 sums of exact products.
template <int DH> constexpr int kParts = DH == 64 ? 1 : 3;
template <int NP>
__device__ __forceinline__ void split8(const f32x16& a, int kk, bf16x8 (&f)[NP]) {
  if constexpr (NP == 1) {
    f[0] = pack8(a, kk);
  } else {
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = a[8 * kk + e];
#pragma unroll
    for (int s = 0; s < NP; ++s) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e)        // the upper halves of two values
        w[e] = __builtin_amdgcn_perm(__builtin_bit_cast(unsigned, r[2 * e + 1]), __builtin_bit_cast(unsigned, r[2 * e]), 0x07060302u);
      f[s] = __builtin_bit_cast(bf16x8, w);
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] -= __builtin_bit_cast(float, __builtin_bit_cast(unsigned, r[e]) & 0xffff0000u);
    }
  }
}
template <int NP>
__device__ __forceinline__ f32x16 mma_parts(const bf16x8& a, const bf16x8 (&f)[NP], f32x16 acc) {
#pragma unroll
  for (int s = NP - 1; s >= 0; --s) acc = MFMA32(a, f[s], acc);      // smallest first
  return acc;
}
// Is any of eight bf16 values infinite or NaN?
__device__ __forceinline__ bool any_non_finite(const bf16x8& v) {
  const u32x4 w = __builtin_bit_cast(u32x4, v);
  bool bad = false;
#pragma unroll
  for (int e = 0; e < 4; ++e) bad = bad || (w[e] & 0x7f80u) == 0x7f80u || (w[e] & 0x7f800000u) == 0x7f800000u;
  return bad;
}
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

// A-operand fragment over a reduction index that is the ROW index of a straight LDS tile s[row][col] (a
// key or query index), for output rows that are its columns c0 .. c0+31 (head-size index): lane (n, hf)
// gets s[r0 + {4hf..4hf+3}][c0 + n] and s[r0 + 8 + {4hf..4hf+3}][c0 + n], the order in which the previous
// MFMA's accumulator holds P / dS.  Done with the transposing LDS read (ds_read_b64_tr_b16): within a
// 16-lane group, lane 4r+c supplies the 8-byte chunk s[row + r][4c..4c+3] and lane 4c+e receives element e
// of the four chunks r = 0..3, so nothing is ever stored transposed.
template <int ALD>
__device__ __forceinline__ bf16x8 frag_tr(const bf16_t (*s)[ALD], int r0, int c0, int lane) {
  const int g = lane >> 4, l16 = lane & 15, hf = g >> 1;
  const bf16_t* p = &s[r0 + 4 * hf + (l16 >> 2)][c0 + 16 * (g & 1) + 4 * (l16 & 3)];
  bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p));
  bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 8 * ALD));
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) { r[e] = lo[e]; r[4 + e] = hi[e]; }
  return r;
}
// A [64 rows][DH cols] bf16 tile (rows r0.., row stride ld, rows >= nrows read as zero) on its way into
// LDS: 256 threads (128 for DH = 16), one or two 16-byte chunks each, held in registers between the global load and
// the LDS store so that the next tile's loads fly while the current tile is computed.
template <int DH>
struct TileRegs {
  static constexpr int NCH = DH == 64 ? 2 : 1, TPR = DH / (8 * NCH);      // chunks per thread, threads per row
  // Decided when compiled: as a run-time test it put a branch around every load and store, and the forward kernel at
  // eight sequences of 1024, 12 heads of 64, took 31.1 us instead of 28.7.
  static constexpr bool ALL = 64 * TPR == 256;
  bf16x8 v[NCH];
  __device__ __forceinline__ void load(const bf16_t* src, size_t ld, int r0, int nrows) {
    const int r = threadIdx.x / TPR, ch = (threadIdx.x % TPR) * 8 * NCH;
#pragma unroll
    for (int i = 0; i < NCH; ++i) v[i] = zero8();
    if ((ALL || r < 64) && r0 + r < nrows) {
      const bf16_t* p = src + (size_t)(r0 + r) * ld + ch;
#pragma unroll
      for (int i = 0; i < NCH; ++i) v[i] = *reinterpret_cast<const bf16x8*>(p + 8 * i);
    }
  }
  // out[r] = the dot product of this tile's row r with the other tile's (fp32; a row's threads are neighbours)
  __device__ __forceinline__ void row_dots(const TileRegs& other, float* out) const {
    const int r = threadIdx.x / TPR;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) s += (float)v[i][e] * (float)other.v[i][e];
#pragma unroll
    for (int x = 1; x < TPR; x <<= 1) s += __shfl_xor(s, x, 64);
    if ((ALL || r < 64) && threadIdx.x % TPR == 0) out[r] = s;
  }
  // Narrow heads: tiles that hold an infinity or a NaN are marked in `bad` (see the tile loops).
  __device__ __forceinline__ void mark(int* bad, int tile) const {
    if constexpr (DH < 64) {
      if (any_non_finite(v[0])) *bad = tile;
    }
  }
  template <int ALD>
  __device__ __forceinline__ void store(bf16_t (*dst)[ALD]) const {
    const int r = threadIdx.x / TPR, ch = (threadIdx.x % TPR) * 8 * NCH;
    if (ALL || r < 64) {
#pragma unroll
      for (int i = 0; i < NCH; ++i) *reinterpret_cast<bf16x8*>(&dst[r][ch + 8 * i]) = v[i];
    }
  }
};

// Narrow heads, tiles with an infinity or a NaN among the rows that P or dS multiplies (or in dS): the sums are then taken
// row by row in fp32, masked rows left out.  In a matrix product a masked row's 0 times infinity, and a zero part of a split
// value times infinity, would be a NaN in outputs that such a row does not reach.
// Score of tile row `row` with this lane column's vector: each half of the wave has eight of every sixteen elements.
template <int NK>
__device__ __forceinline__ float row_dot(const bf16x8 (&f)[NK], const bf16_t* row, int hf) {
  float s = 0.f;
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
#pragma unroll
    for (int e = 0; e < 8; ++e) s = __builtin_fmaf((float)f[kk][e], (float)row[16 * kk + 8 * hf + e], s);
  return s + __shfl_xor(s, 32, 64);
}
template <int ND>
__device__ __forceinline__ void add_row(f32x16 (&acc)[ND], const bf16_t* row, float w, int hf) {
#pragma unroll
  for (int dh = 0; dh < ND; ++dh)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[dh][v] = __builtin_fmaf(w, (float)row[32 * dh + 8 * (v / 4) + 4 * hf + (v % 4)], acc[dh][v]);
}

// Work order.  The grid is one-dimensional: block L takes sequence block L / (B*H) (counted from the heavy end)
// of head-and-batch index L % (B*H).  With causal masking the work of a 128-row block grows with its position
// (shrinks, for the key blocks of dK/dV), and workgroups go to the eight XCDs round-robin by their linear
// index and to compute units as slots free up: so the heaviest blocks start first and the light ones fill the
// gaps, every XCD gets the same mix when B*H is a multiple of 8, and all blocks of one head and batch entry
// run on one XCD, whose L2 then serves their shared K and V (or Q and dO) tiles.
struct AttnBlock { int x, h, b; };
__device__ __forceinline__ AttnBlock attn_block(int index, int H, int BH, int nblk, bool heavy_last) {
  const int cls = index / BH, bh = index % BH;
  AttnBlock a;
  a.x = heavy_last ? nblk - 1 - cls : cls;
  a.h = bh % H;
  a.b = bh / H;
  return a;
}

// P parts: where the blocks of 128 queries (or keys) are few, a block takes 64 or 32 of them, and the two or four waves that share
// them every second or fourth key (query) tile, all brought to LDS together; their partial results are added through LDS.  A
// chain of up to S / 64 tiles becomes one of a half or a quarter, on two or four times as many blocks (measured: see parts_of).
// LDS of a block whose tiles take `tiles` bytes and whose four waves leave `values` partial values a lane over them.
template <int P>
constexpr int sum_bytes(int values, size_t tiles) { return P > 1 && 4 * values * 256 > (int)tiles ? 4 * values * 256 : (int)tiles; }
template <int DH, int P>
struct FwdLds {
  static constexpr int NT = P;
  __attribute__((aligned(16))) bf16_t k[NT][64][kAld<DH>], v[NT][64][kAld<DH>];
  int bad[NT];
  static constexpr int bytes() { return sum_bytes<P>(16 * ((DH + 31) / 32) + 2, sizeof(FwdLds)); }
};
// The waves' partial values, in the memory of the tiles: value i of lane `lane` of wave w at [(w * N + i) * 64 + lane].
template <int N>
__device__ __forceinline__ float& part(float* p, int wave, int i, int lane) { return p[(wave * N + i) * 64 + lane]; }

// ================================================================================= forward
template <int DH, int P>
__global__ void __launch_bounds__(256, P > 1 ? 2 : 3) k_attn_fwd_mfma(const bf16_t* __restrict__ qkv, bf16_t* __restrict__ o,
                                                       float* __restrict__ lse, int S, int H, int BH, int causal) {
  constexpr int NT = P, QB = 128 / P;
  constexpr bool SPLIT = P > 1;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  FwdLds<DH, P>& sm = *reinterpret_cast<FwdLds<DH, P>*>(smem);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, hf = lane >> 5;
  const AttnBlock ab = attn_block(blockIdx.x, H, BH, (S + QB - 1) / QB, causal != 0);
  const int bx = ab.x;
  const int h = ab.h, b = ab.b, d = H * DH;
  constexpr int NK = DH / 16, ND = (DH + 31) / 32, NG = DH >= 32 ? 4 : 2;   // k-steps of a score, output tiles, 8-row groups of one
  const size_t ld = (size_t)3 * d;
  const bf16_t* base = qkv + (size_t)b * S * ld;
  const int q0 = bx * QB + wave / P * 32, slot = wave % P, qi = q0 + n;
  bf16x8 qf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk)
    qf[kk] = qi < S ? *reinterpret_cast<const bf16x8*>(base + (size_t)qi * ld + h * DH + 16 * kk + 8 * hf) : zero8();
  float m = -INFINITY, l = 0.f;
  f32x16 oacc[ND];
#pragma unroll
  for (int dh = 0; dh < ND; ++dh) zero16(oacc[dh]);
  const float c = kScale<DH> * kLog2e;
  int q_hi = bx * QB + QB - 1;
  if (q_hi > S - 1) q_hi = S - 1;
  const int n_tiles = causal ? q_hi / 64 + 1 : (S + 63) / 64;
  TileRegs<DH> kr[NT], vr[NT];
  auto load = [&](int t0) {
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (SPLIT && t0 + u >= n_tiles) break;
      kr[u].load(base + d + h * DH, ld, (t0 + u) * 64, S);
      vr[u].load(base + 2 * d + h * DH, ld, (t0 + u) * 64, S);
    }
  };
  load(0);
  if (DH < 64 && threadIdx.x < NT) sm.bad[threadIdx.x] = -1;
  auto& Ks = sm.k[slot];
  auto& Vs = sm.v[slot];
  for (int t0 = 0; t0 < n_tiles; t0 += NT) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (SPLIT && t0 + u >= n_tiles) break;
      kr[u].store(sm.k[u]);
      vr[u].store(sm.v[u]);
      vr[u].mark(&sm.bad[u], t0 + u);
    }
    __syncthreads();
    const int jt = t0 + slot, k0 = jt * 64;
    const bool slow = DH < 64 && sm.bad[slot] == jt;
    if (t0 + NT < n_tiles) load(t0 + NT);      // the next key tiles' loads fly during these tiles' MFMAs
    const bool active = q0 < S && jt < n_tiles && (!causal || k0 <= q0 + 31);
    if (!active) continue;
    f32x16 st[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      zero16(st[i]);
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Ks[32 * i + n][16 * kk + 8 * hf]);
        st[i] = MFMA32(kf, qf[kk], st[i]);
      }
    }
    // The scale 1/sqrt(DH) * log2(e) is positive: the running maximum is taken over the raw scores and scaled once,
    // and the scaling of every score rides in the fused multiply-add that feeds the exponential.
    float mt = -INFINITY;
    // only tiles that touch the diagonal or the end of the sequence need the mask (wave-uniform test)
    const bool need_mask = k0 + 63 >= S || (causal && k0 + 63 > q0);
    if (need_mask) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          int kj = k0 + 32 * i + 8 * (v / 4) + 4 * hf + (v % 4);
          float s = st[i][v];
          if (kj >= S || (causal && kj > qi)) s = -INFINITY;
          st[i][v] = s;
          mt = fmaxf(mt, s);
        }
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) mt = fmaxf(mt, st[i][v]);
    }
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64)) * c;
    float mn = fmaxf(m, mt);
    float mref = mn == -INFINITY ? 0.f : mn;
    float alpha = exp2f(m - mref);
    float rs = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        float p = __builtin_amdgcn_exp2f(__builtin_fmaf(st[i][v], c, -mref));
        st[i][v] = p;
        rs += p;
      }
    l = l * alpha + rs;
    m = mn;
    // once the running maxima have settled every lane's alpha is exactly 1: skip the rescale then (wave-uniform)
    if (__builtin_amdgcn_ballot_w64(alpha != 1.f) != 0) {
#pragma unroll
      for (int dh = 0; dh < ND; ++dh)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[dh][v] *= alpha;
    }
    if (DH < 64 && slow) {        // key by key
#pragma unroll 1
      for (int r = 0; r < 64 && k0 + r < S; ++r) {
        const float s = row_dot<NK>(qf, Ks[r], hf);
        if (qi >= S || (causal && k0 + r > qi)) continue;
        add_row(oacc, Vs[r], __builtin_amdgcn_exp2f(__builtin_fmaf(s, c, -mref)), hf);
      }
      continue;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        bf16x8 pf[kParts<DH>];
        split8(st[i], kk, pf);
#pragma unroll
        for (int dh = 0; dh < ND; ++dh) oacc[dh] = mma_parts(frag_tr(Vs, 32 * i + 16 * kk, 32 * dh, lane), pf, oacc[dh]);
      }
  }
  float lt = l + __shfl_xor(l, 32, 64);
  if constexpr (SPLIT) {
    constexpr int NV = 16 * ND + 2;
    float* pt = reinterpret_cast<float*>(smem);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16 * ND; ++i) part<NV>(pt, wave, i, lane) = oacc[i / 16][i % 16];
    part<NV>(pt, wave, 16 * ND, lane) = m;
    part<NV>(pt, wave, 16 * ND + 1, lane) = lt;
    __syncthreads();
    float mw[P], M = -INFINITY, L = 0.f;
#pragma unroll
    for (int w = 0; w < P; ++w) { mw[w] = part<NV>(pt, wave - slot + w, 16 * ND, lane); M = fmaxf(M, mw[w]); }
#pragma unroll
    for (int w = 0; w < P; ++w) {
      mw[w] = mw[w] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(mw[w] - M);       // a wave without tiles has no sums
      L += part<NV>(pt, wave - slot + w, 16 * ND + 1, lane) * mw[w];
    }
    if (qi < S) {                              // the waves take the 8-row groups of every output tile by turns
      const float inv = 1.f / L;
      bf16_t* op = o + ((size_t)b * S + qi) * d + h * DH;
#pragma unroll
      for (int dh = 0; dh < ND; ++dh)
#pragma unroll
        for (int x = 0; x < NG; x += P) {
          const int g = x + slot;
          if (NG < P && g >= NG) break;
          bf16x4 r;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < P; ++w) v += part<NV>(pt, wave - slot + w, 16 * dh + 4 * g + j, lane) * mw[w];
            r[j] = (bf16_t)(v * inv);
          }
          *reinterpret_cast<bf16x4*>(op + 32 * dh + 8 * g + 4 * hf) = r;
        }
      if (hf == 0 && slot == 0) lse[((size_t)b * H + h) * S + qi] = (M + log2f(L)) * kLn2;
    }
    return;
  }
  if (qi < S) {
    float inv = 1.f / lt;
    bf16_t* op = o + ((size_t)b * S + qi) * d + h * DH;
#pragma unroll
    for (int dh = 0; dh < ND; ++dh)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        bf16x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = (bf16_t)(oacc[dh][4 * g + j] * inv);
        *reinterpret_cast<bf16x4*>(op + 32 * dh + 8 * g + 4 * hf) = w;
      }
    if (hf == 0) lse[((size_t)b * H + h) * S + qi] = (m + log2f(lt)) * kLn2;
  }
}

// ================================================================================= backward
// LDS of a backward block: its two streamed tiles (K and V, or Q and dO) and, for dK/dV, the rows' statistics.
template <int DH, int P>
struct BwdLds {
  static constexpr int NT = P;
  __attribute__((aligned(16))) bf16_t t0[NT][64][kAld<DH>], t1[NT][64][kAld<DH>];
  __attribute__((aligned(16))) float lse2s[NT][64], deltas[NT][64];
  int bad[NT];
  static constexpr int bytes() { return sum_bytes<P>(32 * ((DH + 31) / 32), sizeof(BwdLds)); }
};

// ---------------------------------------------------------------------------------- dQ (and delta = rowsum(dO * O))
template <int DH, int P>
__device__ __forceinline__ void attn_bwd_dq(const AttnBlock ab, BwdLds<DH, P>& sm, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                            const float* __restrict__ lse, const bf16_t* __restrict__ dout,
                                            bf16_t* __restrict__ dqkv, float* __restrict__ delta, int S, int H, int causal) {
  constexpr int NT = P, QB = 128 / P;
  constexpr bool SPLIT = P > 1;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, hf = lane >> 5;
  const int bx = ab.x;
  const int h = ab.h, b = ab.b, d = H * DH;
  constexpr int NK = DH / 16, ND = (DH + 31) / 32, NG = DH >= 32 ? 4 : 2;   // k-steps of a score, output tiles, 8-row groups of one
  const size_t ld = (size_t)3 * d;
  const bf16_t* base = qkv + (size_t)b * S * ld;
  const int q0 = bx * QB + wave / P * 32, slot = wave % P, qi = q0 + n;
  bf16x8 qf[NK], dof[NK];
  float D = 0.f, lse2 = 0.f;
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    if (qi < S) {
      qf[kk] = *reinterpret_cast<const bf16x8*>(base + (size_t)qi * ld + h * DH + 16 * kk + 8 * hf);
      size_t off = ((size_t)b * S + qi) * d + h * DH + 16 * kk + 8 * hf;
      dof[kk] = *reinterpret_cast<const bf16x8*>(dout + off);
      bf16x8 ov = *reinterpret_cast<const bf16x8*>(o + off);
#pragma unroll
      for (int e = 0; e < 8; ++e) D += (float)dof[kk][e] * (float)ov[e];
    } else {
      qf[kk] = zero8(); dof[kk] = zero8();
    }
  }
  D += __shfl_xor(D, 32, 64);
  if (qi < S) {
    size_t si = ((size_t)b * H + h) * S + qi;
    lse2 = lse[si] * kLog2e;
    if (hf == 0 && slot == 0) delta[si] = D;
  }
  f32x16 dqa[ND];
#pragma unroll
  for (int dh = 0; dh < ND; ++dh) zero16(dqa[dh]);
  const float scale = kScale<DH>, c = scale * kLog2e;
  int q_hi = bx * QB + QB - 1;
  if (q_hi > S - 1) q_hi = S - 1;
  const int n_tiles = causal ? q_hi / 64 + 1 : (S + 63) / 64;
  TileRegs<DH> kr[NT], vr[NT];
  auto load = [&](int t0) {
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (SPLIT && t0 + u >= n_tiles) break;
      kr[u].load(base + d + h * DH, ld, (t0 + u) * 64, S);
      vr[u].load(base + 2 * d + h * DH, ld, (t0 + u) * 64, S);
    }
  };
  if (!SPLIT) load(0);
  if (DH < 64 && threadIdx.x < NT) sm.bad[threadIdx.x] = -1;
  auto& Ks = sm.t0[slot];
  auto& Vs = sm.t1[slot];
  for (int t0 = 0; t0 < n_tiles; t0 += NT) {
    if (SPLIT) load(t0);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (SPLIT && t0 + u >= n_tiles) break;
      kr[u].store(sm.t0[u]);
      vr[u].store(sm.t1[u]);
      kr[u].mark(&sm.bad[u], t0 + u);
    }
    __syncthreads();
    const int jt = t0 + slot, k0 = jt * 64;
    bool slow = DH < 64 && sm.bad[slot] == jt;
    if (!SPLIT && t0 + NT < n_tiles) load(t0 + NT);
    const bool active = q0 < S && jt < n_tiles && (!causal || k0 <= q0 + 31);
    if (!active) continue;
    f32x16 st[2], dp[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      zero16(st[i]); zero16(dp[i]);
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Ks[32 * i + n][16 * kk + 8 * hf]);
        bf16x8 vf = *reinterpret_cast<const bf16x8*>(&Vs[32 * i + n][16 * kk + 8 * hf]);
        st[i] = MFMA32(kf, qf[kk], st[i]);
        dp[i] = MFMA32(vf, dof[kk], dp[i]);
      }
    }
    const bool need_mask = k0 + 63 >= S || q0 + 31 >= S || (causal && k0 + 63 > q0);   // wave-uniform
    if (need_mask) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          int kj = k0 + 32 * i + 8 * (v / 4) + 4 * hf + (v % 4);
          bool masked = kj >= S || qi >= S || (causal && kj > qi);
          float p = __builtin_amdgcn_exp2f(st[i][v] * c - lse2);
          st[i][v] = masked ? 0.f : p * (dp[i][v] - D);
        }
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          float p = __builtin_amdgcn_exp2f(st[i][v] * c - lse2);
          st[i][v] = p * (dp[i][v] - D);        // the factor 1/sqrt(DH) of dS is applied once, to the finished dQ
        }
    }
    if constexpr (DH < 64) {
      float t = 0.f;             // NaN if any dS is not finite
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) t = __builtin_fmaf(st[i][v], 0.f, t);
      slow = slow || __builtin_amdgcn_ballot_w64(t != t) != 0;
      if (slow) {                // key by key
#pragma unroll 1
        for (int r = 0; r < 64 && k0 + r < S; ++r) {
          const float s = row_dot<NK>(qf, Ks[r], hf), dpr = row_dot<NK>(dof, Vs[r], hf);
          if (qi >= S || (causal && k0 + r > qi)) continue;
          add_row(dqa, Ks[r], __builtin_amdgcn_exp2f(s * c - lse2) * (dpr - D), hf);
        }
        continue;
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        bf16x8 dsf[kParts<DH>];
        split8(st[i], kk, dsf);
#pragma unroll
        for (int dh = 0; dh < ND; ++dh) dqa[dh] = mma_parts(frag_tr(Ks, 32 * i + 16 * kk, 32 * dh, lane), dsf, dqa[dh]);
      }
  }
  if constexpr (SPLIT) {
    constexpr int NV = 16 * ND;
    float* pt = reinterpret_cast<float*>(&sm);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i) part<NV>(pt, wave, i, lane) = dqa[i / 16][i % 16];
    __syncthreads();
    if (qi < S) {
      bf16_t* dqp = dqkv + ((size_t)b * S + qi) * ld + h * DH;
#pragma unroll
      for (int dh = 0; dh < ND; ++dh)
#pragma unroll
        for (int x = 0; x < NG; x += P) {
          const int g = x + slot;
          if (NG < P && g >= NG) break;
          bf16x4 r;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < P; ++w) v += part<NV>(pt, wave - slot + w, 16 * dh + 4 * g + j, lane);
            r[j] = (bf16_t)(v * scale);
          }
          *reinterpret_cast<bf16x4*>(dqp + 32 * dh + 8 * g + 4 * hf) = r;
        }
    }
    return;
  }
  if (qi < S) {
    bf16_t* dqp = dqkv + ((size_t)b * S + qi) * ld + h * DH;
#pragma unroll
    for (int dh = 0; dh < ND; ++dh)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        bf16x4 w;
#pragma unroll
        for (int j = 0; j < 4; ++j) w[j] = (bf16_t)(dqa[dh][4 * g + j] * scale);
        *reinterpret_cast<bf16x4*>(dqp + 32 * dh + 8 * g + 4 * hf) = w;
      }
  }
}

// ---------------------------------------------------------------------------------- dK, dV
// OWN_DELTA: a query tile's deltas are taken from its dO and O rows as they come by (a read of O more per key block), so that
// these blocks do not wait for the dQ blocks and both kinds can share a launch.
template <int DH, bool OWN_DELTA, int P>
__device__ __forceinline__ void attn_bwd_dkv(const AttnBlock ab, BwdLds<DH, P>& sm, const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o,
                                             const float* __restrict__ lse, const float* __restrict__ delta,
                                             const bf16_t* __restrict__ dout, bf16_t* __restrict__ dqkv, int S, int H,
                                             int causal) {
  constexpr int NT = P, KB = 128 / P;
  constexpr bool SPLIT = P > 1;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, hf = lane >> 5;
  const int bx = ab.x;
  const int h = ab.h, b = ab.b, d = H * DH;
  constexpr int NK = DH / 16, ND = (DH + 31) / 32, NG = DH >= 32 ? 4 : 2;   // k-steps of a score, output tiles, 8-row groups of one
  const size_t ld = (size_t)3 * d;
  const bf16_t* base = qkv + (size_t)b * S * ld;
  const bf16_t* dob = dout + (size_t)b * S * d;
  const bf16_t* ob = o + (size_t)b * S * d;
  const int k0w = bx * KB + wave / P * 32, slot = wave % P, kj = k0w + n;
  bf16x8 kf[NK], vf[NK];
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    if (kj < S) {
      const bf16_t* kp = base + (size_t)kj * ld + d + h * DH + 16 * kk + 8 * hf;
      kf[kk] = *reinterpret_cast<const bf16x8*>(kp);
      vf[kk] = *reinterpret_cast<const bf16x8*>(kp + d);
    } else {
      kf[kk] = zero8(); vf[kk] = zero8();
    }
  }
  f32x16 dka[ND], dva[ND];
#pragma unroll
  for (int dh = 0; dh < ND; ++dh) { zero16(dka[dh]); zero16(dva[dh]); }
  const float scale = kScale<DH>, c = scale * kLog2e;
  const int t_begin = causal ? (bx * KB) / 64 : 0;
  const int t_end = (S + 63) / 64;
  TileRegs<DH> qr[NT], dor[NT], orow[NT];
  auto load = [&](int t0) {
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (SPLIT && t0 + u >= t_end) break;
      qr[u].load(base + h * DH, ld, (t0 + u) * 64, S);
      dor[u].load(dob + h * DH, (size_t)d, (t0 + u) * 64, S);
      if (OWN_DELTA) orow[u].load(ob + h * DH, (size_t)d, (t0 + u) * 64, S);
    }
  };
  if (!SPLIT) load(t_begin);
  if (DH < 64 && threadIdx.x < NT) sm.bad[threadIdx.x] = -1;
  auto& Qs = sm.t0[slot];
  auto& dOs = sm.t1[slot];
  auto& lse2s = sm.lse2s[slot];
  auto& deltas = sm.deltas[slot];
  const int& bad = sm.bad[slot];
  for (int t0 = t_begin; t0 < t_end; t0 += NT) {
    if (SPLIT) load(t0);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < NT; ++u) {
      if (SPLIT && t0 + u >= t_end) break;
      qr[u].store(sm.t0[u]);
      dor[u].store(sm.t1[u]);
      qr[u].mark(&sm.bad[u], t0 + u);
      dor[u].mark(&sm.bad[u], t0 + u);
      if (OWN_DELTA) dor[u].row_dots(orow[u], sm.deltas[u]);
    }
    if (!SPLIT && t0 + NT < t_end) load(t0 + NT);
    if (threadIdx.x < 64 * NT) {
      const int q = t0 * 64 + threadIdx.x;
      const size_t si = ((size_t)b * H + h) * S + q;
      sm.lse2s[threadIdx.x >> 6][threadIdx.x & 63] = q < S ? lse[si] * kLog2e : 0.f;
      if (!OWN_DELTA) sm.deltas[threadIdx.x >> 6][threadIdx.x & 63] = q < S ? delta[si] : 0.f;
    }
    __syncthreads();
    const int it = t0 + slot, q0 = it * 64;
    const bool active = k0w < S && it < t_end && (!causal || q0 + 63 >= k0w);
    if (!active) continue;
    // the mask matters only where this wave's keys reach the tile's queries or either runs off the end
    const bool need_mask = q0 + 63 >= S || k0w + 31 >= S || (causal && k0w + 31 > q0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      f32x16 s, dp;
      zero16(s); zero16(dp);
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        bf16x8 qa = *reinterpret_cast<const bf16x8*>(&Qs[32 * i + n][16 * kk + 8 * hf]);
        bf16x8 da = *reinterpret_cast<const bf16x8*>(&dOs[32 * i + n][16 * kk + 8 * hf]);
        s = MFMA32(qa, kf[kk], s);
        dp = MFMA32(da, vf[kk], dp);
      }
      // wave-uniform: the masked form only on tiles that touch the diagonal or the end of the sequence
      if (need_mask) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 l4 = *reinterpret_cast<const f32x4*>(&lse2s[32 * i + 8 * g + 4 * hf]);
          f32x4 d4 = *reinterpret_cast<const f32x4*>(&deltas[32 * i + 8 * g + 4 * hf]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            int v = 4 * g + j;
            float p = __builtin_amdgcn_exp2f(s[v] * c - l4[j]);
            int qrow = q0 + 32 * i + 8 * g + 4 * hf + j;
            bool masked = qrow >= S || kj >= S || (causal && kj > qrow);
            p = masked ? 0.f : p;
            s[v] = p;
            dp[v] = p * (dp[v] - d4[j]);
            if constexpr (DH < 64) dp[v] = masked ? 0.f : dp[v];      // also where dO or V is infinite
          }
        }
      } else {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4 l4 = *reinterpret_cast<const f32x4*>(&lse2s[32 * i + 8 * g + 4 * hf]);
          f32x4 d4 = *reinterpret_cast<const f32x4*>(&deltas[32 * i + 8 * g + 4 * hf]);
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            int v = 4 * g + j;
            float p = __builtin_amdgcn_exp2f(s[v] * c - l4[j]);
            s[v] = p;
            dp[v] = p * (dp[v] - d4[j]);          // the factor 1/sqrt(DH) of dS is applied once, to the finished dK
          }
        }
      }
      if constexpr (DH < 64) {
        float t = 0.f;           // NaN if any P or dS is not finite (an infinite P makes its dS infinite or NaN)
#pragma unroll
        for (int v = 0; v < 16; ++v) t = __builtin_fmaf(dp[v], 0.f, t);
        if (bad == it || __builtin_amdgcn_ballot_w64(t != t) != 0) {      // query by query
#pragma unroll 1
          for (int r = 32 * i; r < 32 * i + 32 && q0 + r < S; ++r) {
            const float sr = row_dot<NK>(kf, Qs[r], hf), dpr = row_dot<NK>(vf, dOs[r], hf);
            if (kj >= S || (causal && kj > q0 + r)) continue;
            const float p = __builtin_amdgcn_exp2f(sr * c - lse2s[r]);
            add_row(dva, dOs[r], p, hf);
            add_row(dka, Qs[r], p * (dpr - deltas[r]), hf);
          }
          continue;
        }
      }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        bf16x8 pf[kParts<DH>], dsf[kParts<DH>];
        split8(s, kk, pf);
        split8(dp, kk, dsf);
#pragma unroll
        for (int dh = 0; dh < ND; ++dh) {
          dva[dh] = mma_parts(frag_tr(dOs, 32 * i + 16 * kk, 32 * dh, lane), pf, dva[dh]);
          dka[dh] = mma_parts(frag_tr(Qs, 32 * i + 16 * kk, 32 * dh, lane), dsf, dka[dh]);
        }
      }
    }
  }
  if constexpr (SPLIT) {
    constexpr int NV = 32 * ND;
    float* pt = reinterpret_cast<float*>(&sm);
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16 * ND; ++i) {
      part<NV>(pt, wave, i, lane) = dka[i / 16][i % 16];
      part<NV>(pt, wave, 16 * ND + i, lane) = dva[i / 16][i % 16];
    }
    __syncthreads();
    if (kj < S) {
      bf16_t* dkp = dqkv + ((size_t)b * S + kj) * ld + d + h * DH;
#pragma unroll
      for (int dh = 0; dh < 2 * ND; ++dh)         // dK, then dV
#pragma unroll
        for (int x = 0; x < NG; x += P) {
          const int g = x + slot;
          if (NG < P && g >= NG) break;
          bf16x4 r;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float v = 0.f;
#pragma unroll
            for (int w = 0; w < P; ++w) v += part<NV>(pt, wave - slot + w, 16 * dh + 4 * g + j, lane);
            r[j] = (bf16_t)(dh < ND ? v * scale : v);
          }
          *reinterpret_cast<bf16x4*>(dkp + (dh < ND ? 32 * dh : d + 32 * (dh - ND)) + 8 * g + 4 * hf) = r;
        }
    }
    return;
  }
  if (kj < S) {
    bf16_t* dkp = dqkv + ((size_t)b * S + kj) * ld + d + h * DH;
    bf16_t* dvp = dkp + d;
#pragma unroll
    for (int dh = 0; dh < ND; ++dh)
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        bf16x4 wk, wv;
#pragma unroll
        for (int j = 0; j < 4; ++j) { wk[j] = (bf16_t)(dka[dh][4 * g + j] * scale); wv[j] = (bf16_t)dva[dh][4 * g + j]; }
        *reinterpret_cast<bf16x4*>(dkp + 32 * dh + 8 * g + 4 * hf) = wk;
        *reinterpret_cast<bf16x4*>(dvp + 32 * dh + 8 * g + 4 * hf) = wv;
      }
  }
}

// Both kinds of blocks in one launch, eight of one kind and eight of the other in turn (an XCD gets both, and the heaviest of
// both start first).  Apart, few blocks leave the chip half empty twice: 5 x 511, 7 heads of 64 (140 blocks of a kind)
// 37.2 -> 23.3 us, 2 x 1100, 5 heads 66.4 -> 38.8, 3 x 200, 2 heads 22.1 -> 12.8.  With 512 blocks of a kind, two to a compute
// unit, they are level (64 x 128, 8 heads of 16: 23.0 and 23.4; 4 x 2048, 8 heads of 32: 128 and 120), with more the launches apart win
// (4 x 2048, 16 heads of 64: 163 against 184): one kind's blocks share their tiles in L2.
constexpr int kBwdTogether = 512;
enum BwdKind { BWD_BOTH, BWD_DQ, BWD_DKV };
template <int DH, BwdKind KIND, int P>
__global__ void __launch_bounds__(256, KIND == BWD_DQ ? (DH == 64 ? 2 : 3) : (DH == 16 && P == 1 ? 3 : 2))
k_attn_bwd_mfma(const bf16_t* __restrict__ qkv, const bf16_t* __restrict__ o, const float* __restrict__ lse,
                const bf16_t* __restrict__ dout, bf16_t* __restrict__ dqkv, float* __restrict__ delta, int S, int H, int BH, int causal) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  BwdLds<DH, P>& sm = *reinterpret_cast<BwdLds<DH, P>*>(smem);
  constexpr int RB = 128 / P;
  const int nblk = (S + RB - 1) / RB, n = nblk * BH, n8 = n & ~7, L = blockIdx.x;
  bool dq = KIND == BWD_DQ;
  int index = L;
  if (KIND == BWD_BOTH) {
    if (L < 2 * n8) {
      dq = (L >> 3) & 1;
      index = (L >> 4) * 8 + (L & 7);
    } else {
      const int r = L - 2 * n8;
      dq = r >= n - n8;
      index = n8 + (dq ? r - (n - n8) : r);
    }
  }
  if (KIND != BWD_DKV && dq)
    attn_bwd_dq<DH, P>(attn_block(index, H, BH, nblk, causal != 0), sm, qkv, o, lse, dout, dqkv, delta, S, H, causal);
  else if (KIND != BWD_DQ)
    attn_bwd_dkv<DH, KIND == BWD_BOTH, P>(attn_block(index, H, BH, nblk, false), sm, qkv, o, lse, delta, dout, dqkv, S, H, causal);
}

// Into how many parts a block's chain of tiles is split, n the number of whole blocks.  Alone, us, one / two / four parts:
//            n   S x heads x size     forward               backward
//           12   200 x 2 x 64         7.6   7.6   7.5       13.1    9.6    8.0
//           64  2048 x 4 x 64        33.5  22.7  16.8       61.9   41.4   34.3
//           90  1100 x 5 x 64        20.5  14.6  12.0       40.1   28.6   27.2
//           48   300 x 8 x 64         8.2   7.5   7.5       15.6   12.0   12.6
//           63   300 x 7 x 64         8.3   7.2   7.3       15.6   12.0   12.9
//           64   512 x 8 x 64        11.7   8.9   7.2       20.5   14.3   14.0
//           80   512 x 10 x 64       11.8   9.0   7.9       20.6   16.2   17.8
//           96   300 x 8 x 64         8.2   7.5   7.4       15.4   13.0   15.9
//           96   768 x 8 x 64        15.6  11.3   9.6       27.5   21.3   23.3
//           96  1024 x 12 x 64       19.3  13.6  10.9       34.7   25.8   26.0
//           96  1536 x 8 x 64        26.6  18.1  14.6       48.7   34.4   32.0
//           96   300 x 8 x 32         9.6   8.0   7.7       17.1   13.2   12.8
//           96   512 x 12 x 16       13.1   9.7   7.8       22.2   15.8   15.9
//          126   768 x 7 x 64        15.7  11.6  10.3       30.8   24.2   33.9
//          128  2048 x 8 x 64        34.1  23.0  18.0       64.2   44.4   46.5
//          128   256 x 8 x 64         7.9   7.1   7.2       13.7   11.3   18.2
//          140   511 x 7 x 64        12.0   9.6  11.7       24.7   19.8   33.4
//          243   300 x 9 x 64         8.4   8.1  12.8       19.3   21.3   37.0
//          256  1024 x 8 x 64        19.6  14.8  19.5       37.5   38.1   55.5
//          256   512 x 8 x 32        14.7   9.8  11.9       24.6   24.9   33.5
//          768  1024 x 12 x 64       28.0  31.1  47.5       88.9  112.5  187.1
// Four parts of the backward pass of 64-wide heads are 8 n blocks of both kinds, two to a compute unit: past n = 64 they no longer
// go at once, which only long chains pay back (32 + S / 16, up to 96); the narrower heads' chains are longer.
// Short chains only where the blocks are very few: with another chain's products beside it the chip is not empty, and 128 blocks of
// 256 x 8 x 64 in parts gain nothing (pipelined eight layers of 512: 2039 us in parts, 2009 whole).
static int parts_of(int n, int S, int four, int two) {
  if (S <= 256 ? n > 32 || S <= 64 : n > two) return 1;
  return n <= four && S > 128 ? 4 : 2;
}
int attn_parts(int B, int S, int H, int dh, bool backward) {
  const int n = ((S + 127) / 128) * H * B;
  if (!backward) return parts_of(n, S, 128, 256);
  return parts_of(n, S, dh == 64 && S < 1024 ? 32 + S / 16 : 96, 176);
}

template <int DH, int P>
static hipError_t attn_fwd_t(const OpCtx& c, const void* qkv, void* o, float* lse, int B, int S, int H, int causal) {
  constexpr int QB = 128 / P, lds = FwdLds<DH, P>::bytes();
  if (lds > 64 * 1024) {
    static LdsLimit limit;
    hipError_t e = limit.raise(reinterpret_cast<const void*>(k_attn_fwd_mfma<DH, P>), lds);
    if (e != hipSuccess) return e;
  }
  k_attn_fwd_mfma<DH, P><<<((S + QB - 1) / QB) * H * B, 256, lds, c.stream>>>((const bf16_t*)qkv, (bf16_t*)o, lse, S, H, H * B, causal);
  return hipGetLastError();
}
template <int DH, BwdKind KIND, int P>
static hipError_t attn_bwd_launch(const OpCtx& c, const void* qkv, const void* o, const float* lse, const void* dout,
                                  void* dqkv, float* delta, int B, int S, int H, int causal) {
  constexpr int RB = 128 / P, lds = BwdLds<DH, P>::bytes();
  if (lds > 64 * 1024) {
    static LdsLimit limit;
    hipError_t e = limit.raise(reinterpret_cast<const void*>(k_attn_bwd_mfma<DH, KIND, P>), lds);
    if (e != hipSuccess) return e;
  }
  const int n = ((S + RB - 1) / RB) * H * B;
  k_attn_bwd_mfma<DH, KIND, P><<<KIND == BWD_BOTH ? 2 * n : n, 256, lds, c.stream>>>(
      (const bf16_t*)qkv, (const bf16_t*)o, lse, (const bf16_t*)dout, (bf16_t*)dqkv, delta, S, H, H * B, causal);
  return hipGetLastError();
}
template <int DH>
static hipError_t attn_bwd_t(const OpCtx& c, const void* qkv, const void* o, const float* lse, const void* dout,
                             void* dqkv, float* delta, int B, int S, int H, int causal) {
  const int n = ((S + 127) / 128) * H * B;
  const int parts = c.attn_split ? c.attn_split : attn_parts(B, S, H, DH, true);
  if (parts == 4) return attn_bwd_launch<DH, BWD_BOTH, 4>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal);
  if (parts == 2) return attn_bwd_launch<DH, BWD_BOTH, 2>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal);
  if (n <= kBwdTogether) return attn_bwd_launch<DH, BWD_BOTH, 1>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal);
  hipError_t e = attn_bwd_launch<DH, BWD_DQ, 1>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal);
  return e == hipSuccess ? attn_bwd_launch<DH, BWD_DKV, 1>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal) : e;
}
template <int DH>
static hipError_t attn_fwd_d(const OpCtx& c, const void* qkv, void* o, float* lse, int B, int S, int H, int causal) {
  const int parts = c.attn_split ? c.attn_split : attn_parts(B, S, H, DH, false);
  return parts == 4 ? attn_fwd_t<DH, 4>(c, qkv, o, lse, B, S, H, causal)
                    : (parts == 2 ? attn_fwd_t<DH, 2>(c, qkv, o, lse, B, S, H, causal) : attn_fwd_t<DH, 1>(c, qkv, o, lse, B, S, H, causal));
}
bool attn_mfma_ok(int dh) { return dh == 16 || dh == 32 || dh == 64; }
hipError_t attn_fwd_mfma(const OpCtx& c, const void* qkv, void* o, float* lse, int B, int S, int H, int dh, int causal) {
  if (B * S == 0) return hipSuccess;
  return dh == 64 ? attn_fwd_d<64>(c, qkv, o, lse, B, S, H, causal)
                  : (dh == 32 ? attn_fwd_d<32>(c, qkv, o, lse, B, S, H, causal) : attn_fwd_d<16>(c, qkv, o, lse, B, S, H, causal));
}
hipError_t attn_bwd_mfma(const OpCtx& c, const void* qkv, const void* o, const float* lse, const void* dout,
                         void* dqkv, float* delta, int B, int S, int H, int dh, int causal) {
  if (B * S == 0) return hipSuccess;
  return dh == 64 ? attn_bwd_t<64>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal)
                  : (dh == 32 ? attn_bwd_t<32>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal)
                              : attn_bwd_t<16>(c, qkv, o, lse, dout, dqkv, delta, B, S, H, causal));
}

}  // namespace lp
