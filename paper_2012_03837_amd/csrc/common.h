// Shared declarations of the HIP library: element types, error plumbing, and the internal
// kernel-launch API ("ops") that the layer drivers call.  gfx950 only.
#pragma once
#include <map>
#include <string>

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

namespace lp {

typedef __bf16 bf16_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

enum DType { F32 = 0, BF16 = 1, I32 = 2 };
static inline size_t dtype_size(int dt) { return dt == BF16 ? 2 : 4; }

__device__ __forceinline__ float to_f(float v) { return v; }
__device__ __forceinline__ float to_f(bf16_t v) { return static_cast<float>(v); }
template <typename T> __device__ __forceinline__ T from_f(float f);
template <> __device__ __forceinline__ float from_f<float>(float f) { return f; }
template <> __device__ __forceinline__ bf16_t from_f<bf16_t>(float f) { return static_cast<bf16_t>(f); }

enum Act { ACT_NONE = 0, ACT_RELU = 1, ACT_GELU = 2 };

// GELU in its tanh form, 0.5 x (1 + tanh(u)) with u = c (x + a x^3), written through the identity
// 0.5 (1 + tanh(u)) = sigmoid(2u) = 1 / (1 + e^{-2u}) on the hardware exp2 and reciprocal: absolute error of
// a few 1e-7 and exact limits for large |x| (e^{-2u} = inf gives 0, 0 gives 1).  The library tanhf costs
// several times as many instructions, and in a fused GEMM epilogue the MFMA pipe idles meanwhile.
__device__ __forceinline__ float gelu_gate(float x) {     // sigmoid(2u)
  const float k1 = -2.0f * 0.7978845608028654f * 1.4426950408889634f, k3 = k1 * 0.044715f;
  const float x2 = x * x;
  const float e = __builtin_amdgcn_exp2f(x * (k1 + k3 * x2));          // e^{-2u}
  return __builtin_amdgcn_rcpf(1.0f + e);
}
__device__ __forceinline__ float gelu_f(float x) { return x * gelu_gate(x); }
// d/dx [x s(x)] = s + x s', s' = s (1 - s) 2c (1 + 3 a x^2)
__device__ __forceinline__ float dgelu_f(float x) {
  const float c2 = 2.0f * 0.7978845608028654f, a3 = 3.0f * 0.044715f;
  const float s = gelu_gate(x);
  return s * (1.0f + x * (1.0f - s) * (c2 + c2 * a3 * x * x));
}

// C[M,N] (+)= alpha * sum_k A(m,k) B(n,k), then the epilogue:
//   v = acc (+ bias[n]); if (pre) pre[m,n] = v; v = act(v); if (dact) v *= act'(dact_src[m,n]);
//   if (res) v += res[m,n]; C[m,n] = (accumulate ? C[m,n] : 0) + v.
// A(m,k) = a_kc ? A[m*lda + k] : A[k*lda + m];  B(n,k) = b_kc ? B[n*ldb + k] : B[k*ldb + n].
// Operands, pre, dact_src and res are in the compute dtype; C is compute dtype unless c_f32.
struct GemmArgs {
  const void* A = nullptr; int64_t lda = 0; int a_kc = 1;
  const void* B = nullptr; int64_t ldb = 0; int b_kc = 1;
  void* C = nullptr; int64_t ldc = 0; int c_f32 = 0;
  int M = 0, N = 0, K = 0;
  const float* bias = nullptr;
  int act = ACT_NONE;
  void* pre = nullptr;
  int drop_pre = 0;      // pre is not stored (the kernel is chosen as if it were: the same bits in C)
  const void* dact_src = nullptr; int dact = ACT_NONE; int64_t ldd = 0;
  const void* res = nullptr; int64_t ldr = 0;
  int accumulate = 0;
  // Rows of A / B that exist in memory where that differs from M / N (0: the same).  More than M: an operand stored
  // k-major whose row pitch is padded, so that whole 16-byte chunks can be read past row M.  Fewer than N: the last
  // columns of C are padding, computed from a repeated row.
  int a_rows = 0, b_rows = 0;
  // rowsum[m] (+)= sum_k A(m,k) (A stored k-major): the bias gradient beside a weight gradient
  float* rowsum = nullptr;
};
static inline int rows_of_a(const GemmArgs& g) { return g.a_rows ? g.a_rows : g.M; }
static inline int rows_of_b(const GemmArgs& g) { return g.b_rows ? g.b_rows : g.N; }

// Convolution as an implicit GEMM over NHWC activations and [O,R,S,C] filters.
struct ConvArgs {
  int N, H, W, C;      // input
  int O, R, S;         // filters
  int stride, pad;
  int P, Q;            // output spatial
};

// Optional per-kernel-class timing with HIP events recorded on the launch stream.
enum KernelClass { KC_GEMM = 0, KC_ATTN_FWD, KC_ATTN_BWD, KC_LAYERNORM, KC_SOFTMAX_CE, KC_OPTIMIZER, KC_EMBED,
                   KC_COLSUM, KC_CONV, KC_BATCHNORM, KC_OTHER, KC_GEMM_KERNEL, KC_COUNT };
struct Profiler {
  bool on = false;
  struct Pair { hipEvent_t a, b; int kc; uint64_t tag; const char* kname; double flops; };
  Pair* pairs = nullptr; int cap = 0; int used = 0; int dropped = 0;
  double total_ms[KC_COUNT] = {}; long long launches[KC_COUNT] = {}; double flops[KC_COUNT] = {};
  // GEMM ops by shape: tag = M | N << 20 | K << 40 | a_kc << 60 | b_kc << 61 | c_f32 << 62
  struct ShapeTotal { double ms = 0; long long n = 0; };
  std::map<uint64_t, ShapeTotal> by_shape;
  // Main GEMM kernels by instance name (class KC_GEMM_KERNEL: a pair brackets that one launch, without the
  // partial-sum fix-up an op may launch behind it): launches, summed time, algorithmic FLOPs.
  struct KernelTotal { double ms = 0; long long n = 0; double flops = 0; };
  std::map<std::string, KernelTotal> by_kernel;
};

// Partial sums that a chain of work has left and that one launch adds later (op_add_pending): the parameter gradients of a
// layer's normalisations, which nothing before the update reads, and where they are not taken with its weight gradients its bias
// gradients.  A launch behind another one costs 4.6 us however little it does (what a step of small layers gains; beside the
// products of another chain it waits for a compute unit with sixteen free wave slots: 34 to 193 us for 11 MB, a layer of 768
// over 8192 rows, by how the chains meet), so they too go out with the weight gradients where those are bf16 tiles.
constexpr int kMaxPending = 12;
struct PendingSums {
  float* buf = nullptr;
  size_t cap = 0, used = 0;
  int count = 0;
  struct Sum { const float* part; float* out; int nblk, n, accumulate; } s[kMaxPending];
  // room for `sums` more of `floats` partial sums in all
  float* take(size_t floats, int sums) {
    if (!buf || used + floats > cap || count + sums > kMaxPending) return nullptr;
    float* p = buf + used;
    used += floats;
    return p;
  }
  void add(const float* part, float* out, int nblk, int n, int accumulate) { s[count++] = Sum{part, out, nblk, n, accumulate}; }
};

// Filter gradients whose pieces' sums wait in the split-K workspace until one launch adds them (op_conv_add_pending): nothing
// before the update reads them, and a launch of a few KB costs what any launch costs.  `used` floats of the workspace are taken.
constexpr int kMaxFilters = 8;
struct PendingFilters {
  size_t used = 0;
  int count = 0;
  struct Filter { const float* ws; float* dw; int M, N, splits, accumulate; } f[kMaxFilters];
};

struct OpCtx {
  hipStream_t stream;
  int dt;              // compute dtype
  float* partial;      // fp32 scratch for two-stage reductions
  size_t partial_elems;
  Profiler* prof = nullptr;
  int gemm_variant = 0;         // 0: chosen by the cost model; otherwise a forced GEMM kernel (see lpk_gemm)
  int tile_shape = -1, tile_pieces = 1;   // one-tile-per-block products: a forced tile shape and cut (-1: by the cost model)
  int attn_split = 0;           // attention: a block's chain in 1, 2 or 4 parts (0: by the number of blocks)
  float* splitk_ws = nullptr;   // fp32 workspace for split-K partial sums (may be null: no split-K)
  size_t splitk_elems = 0;
  PendingSums* pending = nullptr;   // where op_layernorm_bwd and op_colsum_batched may leave their sums (null: nowhere)
  PendingFilters* filters = nullptr;   // where op_conv_bwd_weight may leave its pieces (null: nowhere)
  bool with_sums = false;           // op_gemm_grouped: the products' row sums and what is pending go out with their launch
};

// RAII bracket: records an event pair around the launches of one op when profiling is on.
struct ProfScope {
  Profiler* p; hipStream_t s; int idx = -1;
  ProfScope(const OpCtx& c, int kc, double flops = 0.0, uint64_t tag = 0, const char* kname = nullptr)
      : p(c.prof), s(c.stream) {
    if (!p || !p->on) { p = nullptr; return; }
    p->launches[kc] += 1; p->flops[kc] += flops;
    if (p->used >= p->cap) { p->dropped += 1; p = nullptr; return; }
    idx = p->used++;
    p->pairs[idx].kc = kc; p->pairs[idx].tag = tag; p->pairs[idx].kname = kname; p->pairs[idx].flops = flops;
    (void)hipEventRecord(p->pairs[idx].a, s);
  }
  void finish() { if (p) { (void)hipEventRecord(p->pairs[idx].b, s); p = nullptr; } }
  ~ProfScope() { finish(); }
};

// ---- ops (each enqueues on ctx.stream and returns a hipError_t) -------------------------------
hipError_t op_gemm(const OpCtx& c, const GemmArgs& g);
// n independent products in one launch where they qualify (bf16, same reduction length and operand layouts,
// plain fp32 outputs: the weight gradients of one layer), otherwise one after the other.  OpCtx::with_sums: one layer's
// weight gradients, their bias gradients (GemmArgs::rowsum) and its pending sums, the sums in the same launch or ahead of it.
hipError_t op_gemm_grouped(const OpCtx& c, const GemmArgs* gs, int n);
// Whether product g is estimated to be faster in a launch with a group of n (of its reduction and layout) than behind it.
bool gemm_joins(const OpCtx& c, const GemmArgs* group, int n, const GemmArgs& g);
hipError_t op_fill_f32(const OpCtx& c, float* p, size_t n, float v);
// out[0] = <a, b> / (|a| |b|) over n floats (0 if either norm is 0); uses 3 * 128 floats of c.partial
hipError_t op_cosine(const OpCtx& c, const float* a, const float* b, size_t n, float* out);
hipError_t op_copy(const OpCtx& c, const void* src, void* dst, size_t bytes);   // bytes % 16 == 0
hipError_t op_cast_to_compute(const OpCtx& c, const float* src, void* dst, size_t n);
// dst[C][ldd] = src[R][C]^T, bf16, columns R .. ldd - 1 of dst zero; C and ldd multiples of 8, both pointers 16-byte aligned
hipError_t op_transpose_bf16(const OpCtx& c, const void* src, void* dst, int R, int C, int ldd);

hipError_t op_embed_fwd(const OpCtx& c, const int32_t* ids, const float* emb, const float* pe, void* out,
                        int T, int S, int d, int V);
hipError_t op_embed_bwd(const OpCtx& c, const int32_t* ids, const void* dh, float* demb, int T, int V, int d,
                        int accumulate);
hipError_t op_posenc_init(const OpCtx& c, float* pe, int S, int d);

hipError_t op_layernorm_fwd(const OpCtx& c, const void* x, const float* g, const float* b, void* y,
                            float* mean, float* rstd, int rows, int d);
// dx = (add ? add : 0) + LN-backward(dy); dg/db accumulate if `accumulate`.  dx may be null; dg and db may
// both be null (input gradient only).
hipError_t op_layernorm_bwd(const OpCtx& c, const void* dy, const void* x, const float* mean, const float* rstd,
                            const float* g, const void* add, void* dx, float* dg, float* db, int rows, int d,
                            int accumulate);
constexpr int kLnFastRows = 16;      // rows per block, and per partial sum of dg and db, of the vectorised backward kernel
hipError_t op_colsum(const OpCtx& c, const void* dy, int64_t ld, float* out, int rows, int n, int accumulate);
// count (<= 4 for the single pair of launches) column sums over the same rows; the same bits as op_colsum one by one
hipError_t op_colsum_batched(const OpCtx& c, int count, const void* const* dy, const int64_t* ld, float* const* out,
                             int rows, const int* n, int accumulate);

// Adds what is pending, in one launch (the same bits as at once).
hipError_t op_add_pending(const OpCtx& c);

hipError_t op_attn_fwd(const OpCtx& c, const void* qkv, void* o, float* lse, int B, int S, int H, int dh,
                       int causal);
hipError_t op_attn_bwd(const OpCtx& c, const void* qkv, const void* o, const float* lse, const void* dout,
                       void* dqkv, float* delta, int B, int S, int H, int dh, int causal);

// Row-wise softmax cross-entropy over logits z [rows, n] (compute dtype, leading dim ld).
// loss_rows[r] = logsumexp(z_r) - z[r, y_r].  If write_grad: z is overwritten by
// (softmax(z_r) - onehot(y_r)) * inv_rows, and columns n .. pad_to - 1 (pad_to <= ld; 0: none) by zeros.
hipError_t op_softmax_ce(const OpCtx& c, void* z, int64_t ld, const int32_t* y, float* loss_rows, int rows,
                         int n, int write_grad, float inv_rows, int pad_to = 0);
// loss_rows of the logits that product g would store, without storing them; hipErrorInvalidValue (nothing launched) where that
// form does not apply.
hipError_t op_gemm_loss(const OpCtx& c, const GemmArgs& g, const int32_t* y, float* loss_rows);
bool gemm_loss_ok(const OpCtx& c, const GemmArgs& g);      // whether it does
hipError_t op_mean(const OpCtx& c, const float* v, int n, float* out);
// Classifier heads of at most 32 classes on at most 1024 features, up to eight in one launch over the same rows and
// labels: loss_rows, and if `backward` also dZ [rows, ncls] and dfeat = dZ w [rows, in] (and a second copy of it).
struct HeadCe { const void *feat, *w; const float* bias; float* loss_rows; void *dz, *dfeat, *dfeat2; int in, ncls; };
constexpr int kMaxHeads = 8;
struct HeadTable { HeadCe h[kMaxHeads]; int n = 0; };
bool head_ce_ok(int in, int ncls);
hipError_t op_head_ce(const OpCtx& c, const HeadTable& ht, const int32_t* y, int rows, int backward, float inv_rows);

struct OptArgs {
  int kind; float lr, momentum, beta1, beta2, eps, weight_decay; int t; float grad_scale;
};
hipError_t op_optimizer(const OpCtx& c, const OptArgs& o, float* p, const float* g, float* m, float* v,
                        void* p_lowp, size_t n);
// Several ranges [off, off + n) of the same buffers in one launch (offsets and sizes multiples of 4), each with its own
// gradient scale (OptArgs::grad_scale is ignored); the launch also writes out[i][0] = the mean of v[i][0 .. rows) for
// the vectors of a MeanTable, the same bits as op_mean.
constexpr int kMaxOptRanges = 8;
struct OptRanges { size_t off[kMaxOptRanges], n[kMaxOptRanges]; float scale[kMaxOptRanges]; int count = 0; };
struct MeanTable { const float* v[kMaxHeads]; float* out[kMaxHeads]; int rows = 0, count = 0; };
// A matrix [rows][cols] of the buffers (cols a multiple of 8) that is updated with them and whose working copy is also written
// transposed, to t [cols][ldt], columns rows .. ldt - 1 (ldt: rows rounded up to 64) zero.  rows 0: none.
struct OptMatrix { size_t off = 0; int rows = 0, cols = 0, ldt = 0; void* t = nullptr; };
hipError_t op_optimizer_ranges(const OpCtx& c, const OptArgs& o, float* p, const float* g, float* m, float* v, void* p_lowp,
                               const OptRanges& r, const OptMatrix& x, const MeanTable& mt);

hipError_t op_init_normal(const OpCtx& c, float* p, size_t n, float std, uint64_t seed, uint64_t stream_id);

// conv / batchnorm / pooling
// Column statistics of a convolution's output, left by the convolution kernel itself for the batch normalisation
// behind it: for slab t of slab_rows consecutive rows and column j, p = the slab's first row, s0 = sum (z - p),
// s1 = sum (z - p)^2 over the rounded outputs, stored as buf[(0 * nslab + t) * C + j], [(1 * nslab + t) ...] and
// [(2 * nslab + t) ...].  The caller sets buf / cap (floats); nslab stays 0 if the launch did not produce them.
// Used where the normalisation's own statistics are shifted sums as well (bn_shifted: whole 256-thread rows of 8-channel
// chunks, C % 8 == 0); for other channel counts it takes fp64 sums over z, and the convolution leaves none.
static inline bool bn_shifted(int C) { return C >= 8 && 256 % (C / 8) == 0; }
struct ConvStats {
  float* buf = nullptr;
  size_t cap = 0;
  int nslab = 0, slab_rows = 0;
};
hipError_t op_conv_fwd(const OpCtx& c, const ConvArgs& a, const void* x, const void* w, void* out,
                       ConvStats* stats = nullptr);
// dx = data gradient (+ add, an activation-gradient tensor of dx's shape: the other branch of a residual block).
hipError_t op_conv_bwd_data(const OpCtx& c, const ConvArgs& a, const void* dout, const void* w, void* dx,
                            const void* add = nullptr);
hipError_t op_conv_bwd_weight(const OpCtx& c, const ConvArgs& a, const void* dout, const void* x, float* dw,
                              int accumulate);
// Adds what waits in c.filters, in one launch (the same bits as at once).
hipError_t op_conv_add_pending(const OpCtx& c);
// Running statistics of one batch normalisation (the evaluation form of the method appendix B.3 cites).
// use == 0: the forward pass normalises with the batch's statistics and folds them in,
//   mean <- (1 - momentum) mean + momentum mean_B,  var <- (1 - momentum) var + momentum var_B rows / (rows - 1);
// use == 1: it normalises with mean / var as they stand and leaves them alone.
struct BnRunning {
  float* mean = nullptr;
  float* var = nullptr;
  float momentum = 0.f;
  int use = 0;
};
// y = [relu]( bn(z) (+ res) ), batch statistics over rows = N*H*W (or the running ones, see BnRunning);
// saves the mean and reciprocal standard deviation it normalised with.
hipError_t op_batchnorm_fwd(const OpCtx& c, const void* z, const float* g, const float* b, const void* res,
                            void* y, float* mean, float* rstd, int rows, int C, int relu,
                            const BnRunning* run = nullptr, const ConvStats* pre = nullptr);
// dy_eff = relu ? dy * (y > 0) : dy;  dz = bn-backward(dy_eff); dg, db; if dres: dres = dy_eff.
hipError_t op_batchnorm_bwd(const OpCtx& c, const void* dy, const void* y, const void* z, const float* mean,
                            const float* rstd, const float* g, void* dz, void* dres, float* dg, float* db,
                            int rows, int C, int relu, int accumulate);
hipError_t op_avgpool_fwd(const OpCtx& c, const void* x, void* out, int N, int HW, int C);
hipError_t op_avgpool_bwd(const OpCtx& c, const void* dfeat, void* dx, int N, int HW, int C);
hipError_t op_add(const OpCtx& c, const void* a, const void* b, void* out, size_t n);

}  // namespace lp
