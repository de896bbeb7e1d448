// Shared declarations of the gfx950 block library: element types, vector
// loads, wavefront reductions, error plumbing and the internal kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/bigmac_block.h"

namespace bm {

typedef __bf16 bf16_t;

// ---------------------------------------------------------------- errors
void set_error(const char* fmt, ...);
bm_status hip_fail(hipError_t e, const char* what);

#define BM_CHECK_HIP(expr)                                         \
  do {                                                             \
    hipError_t _e = (expr);                                        \
    if (_e != hipSuccess) return ::bm::hip_fail(_e, #expr);        \
  } while (0)

#define BM_CHECK_LAUNCH(name)                                      \
  do {                                                             \
    hipError_t _e = hipGetLastError();                             \
    if (_e != hipSuccess) return ::bm::hip_fail(_e, name);         \
  } while (0)

#define BM_RETURN_IF(st)                                           \
  do {                                                             \
    bm_status _s = (st);                                           \
    if (_s != BM_OK) return _s;                                    \
  } while (0)

#define BM_ARG_CHECK(cond, ...)                                    \
  do {                                                             \
    if (!(cond)) {                                                 \
      ::bm::set_error(__VA_ARGS__);                                \
      return BM_ERR_INVALID_ARG;                                   \
    }                                                              \
  } while (0)

// ---------------------------------------------------------------- profiling
// Optional per-kernel-class timing with HIP events recorded on the launch
// stream (bm_profile_begin / bm_profile_end).  Off: a scope costs one branch.
enum { PROF_GEMM_NT = 0, PROF_GEMM_NN, PROF_GEMM_TN, PROF_ATTN_FWD, PROF_ATTN_BWD, PROF_NORM,
       PROF_ELEMENTWISE, PROF_CLASSES };
struct ProfScope {
  int slot;
  hipStream_t st;
  ProfScope(int cls, double work, hipStream_t stream);
  ~ProfScope();
};

// ---------------------------------------------------------------- device helpers
constexpr int WAVE = 64;

template <typename T> struct Elt;
template <> struct Elt<float> {
  static constexpr int VEC = 4;   // elements per 16-byte access
  __device__ static inline float to_f(float v) { return v; }
  __device__ static inline float from_f(float v) { return v; }
};
template <> struct Elt<bf16_t> {
  static constexpr int VEC = 8;
  __device__ static inline float to_f(bf16_t v) { return (float)v; }
  __device__ static inline bf16_t from_f(float v) { return (bf16_t)v; }
};

// 16-byte vector of elements with float views.
template <typename T> struct alignas(16) Vec16 {
  T v[Elt<T>::VEC];
};

template <typename T>
__device__ inline void load16(const T* p, float (&out)[Elt<T>::VEC]) {
  Vec16<T> t = *reinterpret_cast<const Vec16<T>*>(p);
#pragma unroll
  for (int i = 0; i < Elt<T>::VEC; ++i) out[i] = Elt<T>::to_f(t.v[i]);
}

template <typename T>
__device__ inline void store16(T* p, const float (&in)[Elt<T>::VEC]) {
  Vec16<T> t;
#pragma unroll
  for (int i = 0; i < Elt<T>::VEC; ++i) t.v[i] = Elt<T>::from_f(in[i]);
  *reinterpret_cast<Vec16<T>*>(p) = t;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, WAVE);
  return v;
}

__device__ inline float wave_max(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, WAVE));
  return v;
}

// Phi(z) = (1 + erf(z / sqrt 2)) / 2 and phi(z) = exp(-z^2/2) / sqrt(2 pi) from ONE
// exponential: erfc(x) = (a1 t + ... + a5 t^5) exp(-x^2), t = 1 / (1 + p x), x >= 0
// (Abramowitz & Stegun 7.1.26, absolute error below 1.5e-7, i.e. fp32 rounding level),
// and exp(-x^2) with x = |z| / sqrt 2 is the exponential of the density.
__device__ inline void normal_cdf_pdf(float z, float* cdf, float* pdf) {
  const float x = fabsf(z) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.0f));
  const float e = __builtin_amdgcn_exp2f(-x * x * 1.4426950408889634f);
  float poly = fmaf(t, 1.061405429f, -1.453152027f);
  poly = fmaf(t, poly, 1.421413741f);
  poly = fmaf(t, poly, -0.284496736f);
  poly = fmaf(t, poly, 0.254829592f);
  const float half_erfc = 0.5f * t * poly * e;
  *cdf = z >= 0.f ? 1.0f - half_erfc : half_erfc;
  *pdf = e * 0.39894228040143268f;
}
__device__ inline float gelu_f(float z) {
  float cdf, pdf;
  normal_cdf_pdf(z, &cdf, &pdf);
  return z * cdf;
}

// ---------------------------------------------------------------- host helpers
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int cdiv(long a, long b) { return (int)((a + b - 1) / b); }
inline size_t elt_size(int dtype) { return dtype == BM_DTYPE_BF16 ? 2 : 4; }

// Bump allocator over the caller's workspace; a null base only measures.
struct Arena {
  char* base;
  size_t off = 0;
  explicit Arena(void* b) : base(static_cast<char*>(b)) {}
  template <typename T = void> T* take(size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes, 256);
    return base ? reinterpret_cast<T*>(base + o) : nullptr;
  }
};

// ---------------------------------------------------------------- GEMM
enum { GEMM_NT = 0, GEMM_NN = 1, GEMM_TN = 2 };

// Epilogue of C = acc (+bias) (+residual); all optional.
struct GemmEpilogue {
  const void* bias = nullptr;       // [N] storage dtype
  const void* residual = nullptr;   // [M, ldc] storage dtype
  int out_fp32 = 0;                 // write C as fp32 regardless of dtype (NT/NN)
  // SwiGLU backward fused into the input-gradient GEMM of the down projection (bf16 MFMA path,
  // NN layout): the product dA[M,N] is not stored; with the saved pre-activations
  // up[M, 2N] = [g | u] the epilogue writes d_up[M, 2N] = [dA u silu'(g) | dA silu(g)] and the
  // activation a[M,N] = silu(g) u (which the weight-gradient GEMM of the down projection reads).
  const void* swiglu_up = nullptr;  // [M, 2N] storage dtype, row stride 2N
  void* swiglu_dup = nullptr;       // [M, 2N]
  void* swiglu_a = nullptr;         // [M, N]
  // SwiGLU forward fused into the up projection (bf16 MFMA path, NT layout, no bias, N a multiple of
  // 256): C[M, N] = [g | u] is written as usual and the epilogue also writes the activation
  // a[M, N/2] = silu(g) u, taken from the ROUNDED g and u (what a separate pass over C would read).
  // A tile gathers its weight rows from both halves, so that g and u of a column meet in one wavefront.
  void* swiglu_fwd_a = nullptr;     // [M, N/2]
  // GELU in the epilogue, where gemm_fuses_gelu() says so (C contiguous): few fp32 rows.
  // NT: gelu_a[M, N] = gelu(C).
  void* gelu_a = nullptr;
  // NN: dA[M, N] is not stored; gelu_dup = dA gelu'(up), gelu_act = gelu(up) and, with gelu_sums, the column sums of
  // every 16 rows of gelu_dup: [cdiv(M, 16), N]
  const void* gelu_up = nullptr;
  void *gelu_dup = nullptr, *gelu_act = nullptr;
  float* gelu_sums = nullptr;
};

// gemm_scratch_bytes: what a product can make use of; NT and NN also run in less, TN and the generic
// back end need gemm_scratch_need().  TN: grows with K only.
size_t gemm_scratch_bytes(int layout, int M, int N, int K, int dtype);
size_t gemm_scratch_need(int layout, int M, int N, int K, int dtype);
// workspace of a TN product of up to M rows (of C); grows with M
size_t gemm_tn_scratch_rows(int M, int N, int K, int dtype);
// workspace of the NT / NN products of up to `rows` rows and N columns: their k ranges are split only
// while splits x rows stays below SPLIT_ROWS_MAX (few rows leave the chip idle otherwise).  Grows with
// `rows`, so that a buffer sized for the longest pack serves every shorter one.
constexpr int SPLIT_ROWS_MAX = 4096;
inline size_t gemm_rows_scratch_bytes(int rows, int N, int dtype) {
  if (dtype != BM_DTYPE_BF16) return 0;
  const long r = (long)rows * 16 < SPLIT_ROWS_MAX ? (long)rows * 16 : SPLIT_ROWS_MAX;
  return (size_t)r * N * sizeof(float);
}
bm_status gemm(int layout, int dtype, int M, int N, int K, const void* A, int lda, const void* B,
               int ldb, void* C, int ldc, const GemmEpilogue& epi, void* scratch,
               size_t scratch_bytes, hipStream_t st);

// contiguous rows, 16-byte aligned operands
bool gemm_fuses_gelu(int layout, int dtype, int M, int N, int K);

// An input gradient C[M,N] = A[M,K] B[K,N] and a weight gradient C[M,N] += A[K,M]^T B[K,N] (fp32 C) that do not depend on
// one another: one launch where few rows leave the chip idle, else one after the other.  Scratch as for both.
struct GemmCall { int M, N, K; const void* A; int lda; const void* B; int ldb; void* C; int ldc; };
bm_status gemm_nn_tn(int dtype, const GemmCall& nn, const GemmCall& tn, void* scratch, size_t scratch_bytes, hipStream_t st);
// one launch, with its status in *rc; or false and nothing launched: separate launches are the better choice
bool gemm_nn_tn_joint(int dtype, const GemmCall& nn, const GemmCall& tn, void* scratch, size_t scratch_bytes, hipStream_t st,
                      bm_status* rc);
// room for both, given what either is given on its own
size_t gemm_nn_tn_scratch_bytes(size_t nn, size_t tn, int dtype);
bool gemm_mfma_nn_tn(const GemmCall& nn, const GemmCall& tn, void* scratch, size_t scratch_bytes, hipStream_t st, bm_status* rc);
bool gemm_generic_nn_tn_shares(int dtype, const GemmCall& nn, const GemmCall& tn);
// the k ranges of either where they share a launch, else 0
void gemm_nn_tn_ranges(int dtype, const GemmCall& nn, const GemmCall& tn, size_t scratch_bytes, int* nn_ranges, int* tn_ranges);
bool gemm_mfma_nn_tn_ranges(const GemmCall& nn, const GemmCall& tn, size_t scratch_bytes, int* nn_ranges, int* tn_ranges);
bool gemm_generic_nn_tn(int dtype, const GemmCall& nn, const GemmCall& tn, hipStream_t st, bm_status* rc);

// Grouped GEMM for the mixture-of-experts FFN: the rows of the activation matrices are
// sorted by expert and every expert's segment is padded to MOE_PAD rows.
//   NT / NN: row block t (MOE_PAD rows) of A and C belongs to group tile_group[t] (-1: no
//            group, the block is skipped); the B matrix of group g starts at B + g*b_stride.
//   TN:      group g contracts over rows [group_rows[g], group_rows[g+1]) of A and B and
//            accumulates into the fp32 matrix at C + g*c_stride.
// M (NT/NN) resp. K (TN) is the padded row capacity, a multiple of MOE_PAD.
constexpr int MOE_PAD = 128;
struct GemmGroups {
  const int32_t* tile_group = nullptr;   // dev [rows / MOE_PAD]     (NT, NN)
  const int32_t* group_rows = nullptr;   // dev [n_groups + 1]       (TN)
  const int32_t* row_tiles = nullptr;    // dev [1 + row_tiles_cap]  (NT, NN): their number, then for each twice its first row block,
  int row_tiles_cap = 0;                 //   plus one where it holds the next block of the same group as well
  // Rows read where they lie instead of from a sorted copy (gemm_mfma_reads_source_rows): the source row, of src_rows, of each row of A
  // (NT, NN) or of each k row of A (source_operand 0) or B (1) (TN, src_rows at most MOE_SOURCE_ROWS).  A source row stands at
  // most once in a group.  Rows without one stand at the end of a group: they read some row of it (NT, NN: results that are
  // never read; TN: they add nothing).
  const int32_t* source = nullptr;
  int src_rows = 0, source_operand = 0;
  const float* row_scale = nullptr;      // dev [rows]: factor of every row of A, with the SwiGLU backward epilogue (its activation included)
  float* row_dot = nullptr;              // dev [rows, N / 64] with it: what the row's product with the activation sums to, without the factor
  int n_groups = 0;
  long b_stride = 0;                     // elements between the B matrices of two groups (NT, NN)
  long c_stride = 0;                     // elements between the C matrices of two groups (TN)
  long routed_rows = 0;                  // rows that carry tokens (profiling: algorithmic flops)
};
// Two weight gradients over the same rows, C_i[M_i,N_i] += A_i[K,M_i]^T B_i[K,N_i] (fp32 C), as one
// launch when that fills the chip better, else one after the other; scratch as for the larger sum
// of both (gemm_pair_scratch_bytes).
size_t gemm_tn_pair_scratch_bytes(int K, int M0, int N0, int M1, int N1, int dtype);
bm_status gemm_tn_pair(int dtype, int K, int M0, int N0, const void* A0, int lda0, const void* B0, int ldb0,
                       void* C0, int ldc0, int M1, int N1, const void* A1, int lda1, const void* B1, int ldb1,
                       void* C1, int ldc1, void* scratch, size_t scratch_bytes, hipStream_t st);
bool gemm_tn_pair_shares_launch(int dtype, int K, int M0, int N0, const void* A0, int lda0, const void* B0, int ldb0,
                                void* C0, int ldc0, int M1, int N1, const void* A1, int lda1, const void* B1, int ldb1,
                                void* C1, int ldc1, void* scratch, size_t scratch_bytes, hipStream_t st);
size_t gemm_mfma_tn_pair_scratch_bytes(int K, int M0, int N0, int M1, int N1);
bool gemm_mfma_tn_pair(int K, int M0, int N0, const void* A0, int lda0, const void* B0, int ldb0, void* C0, int ldc0,
                       int M1, int N1, const void* A1, int lda1, const void* B1, int ldb1, void* C1, int ldc1,
                       void* scratch, size_t scratch_bytes, hipStream_t st, bm_status* rc, double* time = nullptr);
// All weight gradients of a block (the same rows, at most 4) in one launch; scratch as for any of them alone.  `pays`:
// expected to be faster than launches that follow one another, where nn[i] and tn[i] (i < 2: up/down, o/up) can share
// one and so can either nn[2] and tn[2] (qkv/o) or tn[2] and tn[3] (o/qkv); the second form: where none of them do.
bool gemm_tn_group_pays(int dtype, const GemmCall nn[3], const GemmCall tn[4], size_t scratch_bytes);
bool gemm_tn_group_pays(int dtype, const GemmCall* tn, int n, size_t scratch_bytes);
bm_status gemm_tn_group(const GemmCall* tn, int n, void* scratch, size_t scratch_bytes, hipStream_t st);
bm_status gemm_mfma_tn_group(const GemmCall* tn, int n, void* scratch, size_t scratch_bytes, hipStream_t st);
// the k ranges of each where they share that launch (host only), and of either of a pair that shares one
void gemm_mfma_tn_group_ranges(const GemmCall* tn, int n, size_t scratch_bytes, int32_t* k_ranges);
int gemm_mfma_tn_pair_ranges(int K, int M0, int N0, int M1, int N1);
// expected times in us; < 0: not supported or not the choice
double gemm_mfma_tn_group_time(const GemmCall* tn, int n, size_t scratch_bytes);
double gemm_mfma_nn_tn_time(const GemmCall& nn, const GemmCall& tn, size_t scratch_bytes);
double gemm_mfma_time(int layout, const GemmCall& w, size_t scratch_bytes);
// epi (MFMA path only, the caller checks gemm_mfma_grouped_supported): the SwiGLU epilogues of
// GemmEpilogue, forward on NT (N a multiple of 256) and backward on NN (N a multiple of 256)
bm_status gemm_grouped(int layout, int dtype, int M, int N, int K, const void* A, int lda,
                       const void* B, int ldb, void* C, int ldc, const GemmGroups& g, hipStream_t st,
                       const GemmEpilogue* epi = nullptr);
constexpr int MOE_SOURCE_ROWS = 8192;
bool gemm_mfma_reads_source_rows(int layout, int M, int N, const GemmEpilogue* epi);
bool gemm_mfma_grouped_supported(int layout, int dtype, int M, int N, int K, int lda, int ldb, int ldc);
bm_status gemm_mfma_grouped(int layout, int M, int N, int K, const void* A, int lda, const void* B,
                            int ldb, void* C, int ldc, const GemmGroups& g, hipStream_t st,
                            const GemmEpilogue* epi = nullptr);
bm_status gemm_generic_grouped(int layout, int dtype, int M, int N, int K, const void* A, int lda,
                               const void* B, int ldb, void* C, int ldc, const GemmGroups& g,
                               hipStream_t st);

// ---------------------------------------------------------------- mixture of experts
// Device tables of one routed batch (all caller memory, see moe.hip for the layout).
struct MoeTables {
  int cap = 0;                 // padded row capacity, moe_row_capacity(T, E, k)
  float* probs = nullptr;      // [T, E] router probabilities
  int32_t* idx = nullptr;      // [T, k] chosen experts, by descending probability
  float* gate = nullptr;       // [T, k] normalised gates
  int32_t* slot = nullptr;     // [T, k] row of each choice in the expert-sorted layout
  int32_t* row_token = nullptr;   // [cap] token of a row, -1 for padding
  float* row_gate = nullptr;      // [cap] gate of a row
  int32_t* tile_group = nullptr;  // [cap / MOE_PAD] expert of a row block, -1 past the end
  int32_t* expert_rows = nullptr; // [E + 1] padded segment offsets
  int32_t* row_tiles = nullptr;   // [1 + moe_row_tiles_cap] see GemmGroups
};
int moe_row_capacity(int T, int E, int k);
inline int moe_row_tiles_cap(int cap, int E) { return (cap / MOE_PAD + E) / 2; }
size_t moe_layout_scratch_bytes(int T, int E);
bm_status moe_check(int E, int k, int d, int dtype);
bm_status moe_route(const float* logits, int T, int E, int k, float* probs, int32_t* idx, float* gate,
                    hipStream_t st);
bm_status moe_layout(const MoeTables& m, int T, int E, int k, void* scratch, hipStream_t st);
bm_status moe_gather(int dtype, const void* src, const MoeTables& m, int use_gate, void* dst, int d, int T,
                     hipStream_t st);
bm_status moe_combine(int dtype, const void* rows, const MoeTables& m, int use_gate, const void* res,
                      void* out, int T, int k, int d, hipStream_t st);
// the gradient of a gate is <dm, y_rows> of its routed row, or the sum of the row's `parts` values of row_dot (then dm and y_rows are
// not read)
bm_status moe_router_backward(int dtype, const void* dm, const void* y_rows, const float* row_dot, int parts, const MoeTables& m,
                              void* dlogits, int T, int E, int k, int d, hipStream_t st);

// generic (any shape, fp32 arithmetic) and MFMA (bf16) back ends
size_t gemm_generic_scratch_bytes(int M, int N, int K);
bm_status gemm_generic(int layout, int dtype, int M, int N, int K, const void* A, int lda,
                       const void* B, int ldb, void* C, int ldc, const GemmEpilogue& epi,
                       void* scratch, size_t scratch_bytes, hipStream_t st);
bool gemm_mfma_supported(int layout, int dtype, int M, int N, int K, int lda, int ldb, int ldc,
                         const GemmEpilogue& epi);
size_t gemm_mfma_scratch_bytes(int layout, int M, int N, int K);
void gemm_mfma_plan(int layout, int M, int N, int K, size_t scratch_bytes, int* bm, int* bn, int* splits);
bm_status gemm_mfma(int layout, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                    void* C, int ldc, const GemmEpilogue& epi, void* scratch, size_t scratch_bytes,
                    hipStream_t st);

// ---------------------------------------------------------------- attention
struct AttnArgs {
  int dtype, causal, Hq, Hkv, dh;
  const void *q, *k, *v;   // row stride ld_qkv elements
  int ld_qkv;
  const int32_t* cu_dev;
  const int32_t* cu_host;
  int S, T, max_seqlen;
  // Keys/values packed on their own (one chunk of a context-parallel partition of the same S
  // sequences): offsets, rows, row stride and longest segment.  cu_k_dev == nullptr: they share
  // the queries' packing and row stride.  Under a causal mask both packings must be equal (the
  // chunk attends to itself).  ld_dkv: row stride of dk/dv when it differs from dq's.
  const int32_t* cu_k_dev = nullptr;
  const int32_t* cu_k_host = nullptr;
  int Tk = 0, ld_kv = 0, max_klen = 0, ld_dkv = 0;
  // backward: a gradient lies in memory that an input takes up (set by attention_backward).  dK/dV and dQ tiles then do not
  // run side by side: either would read what the other has already overwritten.
  bool in_place = false;
  const int32_t* kv_cu_dev() const { return cu_k_dev ? cu_k_dev : cu_dev; }
  const int32_t* kv_cu_host() const { return cu_k_dev ? cu_k_host : cu_host; }
  int kv_T() const { return cu_k_dev ? Tk : T; }
  int kv_ld() const { return cu_k_dev ? ld_kv : ld_qkv; }
  int kv_max_len() const { return cu_k_dev ? max_klen : max_seqlen; }
};
bm_status attention_forward(const AttnArgs& a, void* o, float* lse, hipStream_t st);
size_t attention_backward_scratch_bytes(int Hq, int Hkv, int dh, int T);
size_t attention_backward_scratch_bytes(int Hq, int Hkv, int dh, int Tq, int Tk);
bm_status attention_backward(const AttnArgs& a, const void* o, const void* d_o, const float* lse,
                             void* dq, void* dk, void* dv, int ld_dqkv, void* scratch,
                             size_t scratch_bytes, hipStream_t st);

bm_status attention_forward_generic(const AttnArgs& a, void* o, float* lse, hipStream_t st);
bm_status attention_backward_generic(const AttnArgs& a, const void* o, const void* d_o,
                                     const float* lse, void* dq, void* dk, void* dv, int ld_dqkv,
                                     float* delta, hipStream_t st);

// ---------------------------------------------------------------- elementwise / norms
// seq id of every token: tok_seq[t] = s with cu[s] <= t < cu[s+1]
bm_status launch_tok_seq(const int32_t* cu_dev, int S, int T, int32_t* tok_seq, hipStream_t st);

// Column sums that kernels have left as partial rows in scratch (bias and gain gradients); one launch folds all of a
// list into their fp32 accumulators.  Scratch that a target points to stays untouched until the flush.
struct ColumnSums {
  static constexpr int MAX = 16;
  struct Target { const float* partial; float* out; int parts, stride, n; } target[MAX];
  int count = 0;
  // out[c] += sum over p < parts of partial[p * stride + c], c < n
  bm_status add(const float* partial, int parts, int stride, int n, float* out) {
    if (count == MAX) { set_error("more than %d column sums in one list", MAX); return BM_ERR_INVALID_ARG; }
    target[count++] = Target{partial, out, parts, stride, n};
    return BM_OK;
  }
};
bm_status flush_column_sums(ColumnSums* sums, hipStream_t st);

// The same for the per-sequence sums of the adaLN gradients whose rows are shared by several workgroups: the flush writes
// out[s, off_q + n] = sum over r < parts of partial[s, r, q, n].
struct SegmentSums {
  static constexpr int MAX = 8;
  struct Target { const float* partial; float* out; int S, parts, planes, N, ld_out, off0, off1; } target[MAX];
  int count = 0;
  bm_status add(const Target& t) {
    if (count == MAX) { set_error("more than %d segment sums in one list", MAX); return BM_ERR_INVALID_ARG; }
    target[count++] = t;
    return BM_OK;
  }
};
bm_status flush_segment_sums(SegmentSums* sums, hipStream_t st);

struct NormArgs {
  int dtype, kind;          // BM_NORM_*
  int T, d;
  float eps;
  const void* gamma = nullptr;
  const void* beta = nullptr;
  const float* mod = nullptr;        // adaLN: fp32 [S, ld_mod]
  int ld_mod = 0, shift_off = 0, scale_off = 0;
  const int32_t* tok_seq = nullptr;
};
// h = N(x); stats[2T] = (mean, rstd) written when write_stats
bm_status norm_forward(const NormArgs& a, const void* x, void* h, float* stats, int write_stats,
                       hipStream_t st);
// sums: with dsum_res and dsum_out
size_t norm_backward_scratch_bytes(int kind, bool sums, int T, int d);
// dx = dres + dN/dx(dh);  dgamma/dbeta fp32 += (LayerNorm/RMSNorm) and dsum_res/dsum_out when `sums` is flushed
// adaLN: dmod[:, shift_off..] = segsum(dh), dmod[:, scale_off..] = segsum(dh * xhat) (overwrite, fp32), whole when
// `segments` is flushed (null otherwise)
bm_status norm_backward(const NormArgs& a, const void* x, const float* stats, const void* dh,
                        const void* dres, void* dx, void* h_out, float* dgamma, float* dbeta,
                        float* dsum_res, float* dsum_out, float* dmod, const int32_t* cu_dev, int S,
                        void* scratch, ColumnSums* sums, SegmentSums* segments, hipStream_t st);

// RoPE in place on the first n_heads heads of each row of qkv; sign=+1 fwd, -1 bwd
bm_status rope_inplace(int dtype, void* qkv, int ld, int T, int n_heads, int dh, float base,
                       const int32_t* cu_dev, const int32_t* tok_seq, float sign, hipStream_t st);

bm_status act_forward(int dtype, int act, const void* up, void* a, int T, int F, hipStream_t st);
bm_status act_backward(int dtype, int act, const void* up, const void* da, void* dup, void* a_out,
                       float* bias_grad, void* scratch, int T, int F, ColumnSums* sums, hipStream_t st);

// out[n] += sum_t a[t, n]   (fp32 accumulate, deterministic two-stage; the second stage is the list's flush)
size_t colsum_scratch_bytes(int T, int N);
bm_status colsum_accumulate(int dtype, const void* a, int lda, int T, int N, float* out,
                            void* scratch, ColumnSums* sums, hipStream_t st);
// out[s, n] = sum_{t in s} a[t,n] * b[t,n] (fp32, overwrite) and, when gated != nullptr,
// gated[t, n] = a[t, n] * gate[s, n]; rows are N wide; scratch: segment_scratch_bytes(), until `sums` is flushed.
// bias_grad (nullable): += the column sums of gated when `columns` is flushed, with columns_ws until then
// (segment_columns_bytes() and colsum_scratch_bytes(T, N), the larger)
size_t segment_scratch_bytes();
size_t segment_columns_bytes();
bm_status segment_gate(int dtype, const void* a, const void* b, const float* gate, int ld_gate, void* gated,
                       const int32_t* cu_dev, int S, int T, int N, float* out, int ld_out, void* scratch,
                       SegmentSums* sums, float* bias_grad, void* columns_ws, ColumnSums* columns, hipStream_t st);
// out[t, n] = (residual ? residual[t,n] : 0) + a[t, n] * gate[tok_seq[t], n]
bm_status gate_mul(int dtype, const void* a, const float* gate, int ld_gate,
                   const int32_t* tok_seq, const void* residual, void* out, int T, int N,
                   hipStream_t st);
// out = silu(in) (storage dtype) ; dsilu: out = g * silu'(in) with g fp32
bm_status silu_forward(int dtype, const void* in, void* out, long n, hipStream_t st);
bm_status silu_backward_f32(int dtype, const void* in, const float* g, void* out, long n,
                            hipStream_t st);
// operands of the adaLN projection's backward from dmod [S, W] and cond [S, d]: e, t (transposed, S8 >= S columns), sc (nullable)
// and the cleared accumulator acc [S8, d]; W >= d
bm_status ada_operands(int dtype, const float* dmod, const void* cond, void* e, void* t, void* sc, float* acc, int S, int S8,
                       int W, int d, hipStream_t st);

}  // namespace bm

// ---------------------------------------------------------------- handoff (executor)
namespace bm {
bm_status row_scatter(int dtype, const void* src, const int32_t* rows, void* dst, int n, int width, hipStream_t st);
bm_status row_gather(int dtype, const void* src, const int32_t* rows, void* dst, int n, int width, hipStream_t st);
bm_status fill_zero(void* p, size_t bytes, hipStream_t st);
bm_status add_inplace(int dtype, void* a, const void* b, long n, hipStream_t st);
size_t loss_scratch_bytes();
// grad = (out - target)/n, *loss = 0.5 * mean((out - target)^2)
bm_status mse_loss(int dtype, const void* out, const void* target, void* grad, long n, float* loss, void* scratch, hipStream_t st);
// *loss = <out, g>
bm_status dot_loss(int dtype, const void* out, const void* g, long n, float* loss, void* scratch, hipStream_t st);
}  // namespace bm
