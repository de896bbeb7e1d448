// Shape-agnostic GEMM with fp32 arithmetic.  It is the fp32 check path of
// the block and the cover for shapes the bf16 MFMA kernels do not take (tiny or
// oddly sized problems such as the adaLN conditioning projection).
//
//   NT: C[M,N]  = A[M,K] B[N,K]^T      NN: C[M,N] = A[M,K] B[K,N]
//   TN: C[M,N] += A[K,M]^T B[K,N]      (C fp32, accumulated)
//
// Operands go from memory straight into the registers of v_mfma_f32_16x16x4_f32: no LDS, no barrier
// in the loop, and many loads in flight.  The small products this serves are bound by latency, and
// the 64x64 LDS tiles that were here paid one memory latency, two barriers and 16 rounds of LDS
// reads per 16 k: NT 40x64x256 27.5 -> 8.2 us (the launch itself), 1024x256x256 29.6 -> 8.3,
// 256x64x1000 96 -> 8.5, 1000x1000x1000 118 -> 36, 2048x2048x2048 461 -> 157, 4096x4096x1024 927 -> 355
// (TN 526 -> 391).  Error against fp64 as before, half of it where four wavefronts share a k range.
// Every access is clamped into its matrix; what lies past the k range counts as zero.
#include "common.h"

namespace bm {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NUM_CU = 256;
constexpr int GT = 64;   // tile edge the k split is chosen for
constexpr int GK = 16;   // k step: four MFMAs; lane l holds k = 4 (l/16) + s of step s

// Operand values of one 16(row) x 16(k) block: lane l has row l%16, v[s] is k = k0 + 4 (l/16) + s.
// KCONT: k is contiguous in memory (row stride ld), else rows are (k stride ld).  WIDE: the four values
// of a lane are one aligned load, and the k range ends on a multiple of 4.
template <typename T, bool KCONT, bool WIDE>
__device__ inline void load_block(const T* __restrict__ p, int ld, int row, int rows, int k0, int kfin, int lane,
                                  float (&v)[4]) {
  const int r = min(row + (lane & 15), rows - 1), k = k0 + (lane >> 4) * 4;
  if (KCONT && WIDE) {
    struct alignas(4 * sizeof(T)) Four { T e[4]; };
    const Four f = *reinterpret_cast<const Four*>(p + (size_t)r * ld + min(k, kfin - 4));
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = k < kfin ? Elt<T>::to_f(f.e[s]) : 0.f;
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int kc = min(k + s, kfin - 1);
      const float x = Elt<T>::to_f(KCONT ? p[(size_t)r * ld + kc] : p[(size_t)kc * ld + r]);
      v[s] = k + s < kfin ? x : 0.f;
    }
  }
}

// F = 1: a workgroup owns one 16x16 tile and its four wavefronts take every fourth k step each; the
// four sums meet in LDS.  F = 2, 4: a wavefront owns F x F blocks, a workgroup 32F x 32F.
// With k_per_split < K the grid's z index selects a k range and the workgroup stores
// its fp32 partial tile into `partial` [z][M][N]; finish_kernel then sums the ranges
// in order and applies the epilogue (skinny problems: few output tiles, long K).
template <typename T, int LAYOUT, int F, bool WIDE>
__global__ __launch_bounds__(256) void gemm_generic_kernel(
    int M, int N, int K, const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
    void* __restrict__ Cv, int ldc, const T* __restrict__ bias, const T* __restrict__ residual,
    int out_fp32, int k_per_split, float* __restrict__ partial, GemmGroups grp) {
  constexpr int TILE = F == 1 ? 16 : 32 * F;
  constexpr bool A_KCONT = LAYOUT != GEMM_TN, B_KCONT = LAYOUT == GEMM_NT;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m_tile = blockIdx.y * TILE, n_tile = blockIdx.x * TILE;
  int kbeg = blockIdx.z * k_per_split;
  int kfin = min(K, kbeg + k_per_split);
  if (grp.group_rows) {              // grouped weight gradient: blockIdx.z is the group
    kbeg = min(grp.group_rows[blockIdx.z], K);
    kfin = min(grp.group_rows[blockIdx.z + 1], K);
    if (kbeg >= kfin) return;
    Cv = (float*)Cv + (long)blockIdx.z * grp.c_stride;
  } else if (grp.tile_group) {       // grouped forward / input gradient: B of this row block's group
    const int g = grp.tile_group[m_tile / MOE_PAD];
    if (g < 0) return;
    B += (long)g * grp.b_stride;
  }
  auto store = [&](int gm, int gn, float v) {
    if (gm >= M || gn >= N) return;
    const size_t idx = (size_t)gm * ldc + gn;
    if (partial) {
      partial[((size_t)blockIdx.z * M + gm) * N + gn] = v;
    } else if (LAYOUT == GEMM_TN) {
      ((float*)Cv)[idx] += v;
    } else {
      if (bias) v += Elt<T>::to_f(bias[gn]);
      if (residual) v += Elt<T>::to_f(residual[idx]);
      if (out_fp32) ((float*)Cv)[idx] = v;
      else ((T*)Cv)[idx] = Elt<T>::from_f(v);
    }
  };
  const int col = lane & 15, row4 = (lane >> 4) * 4;      // accumulator: column, first of four rows
  if constexpr (F == 1) {
    constexpr int DEPTH = 4;         // k steps of a wavefront in flight
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int k0 = kbeg + wave * GK; k0 < kfin; k0 += DEPTH * 4 * GK) {
      float a[DEPTH][4], b[DEPTH][4];
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        load_block<T, A_KCONT, WIDE>(A, lda, m_tile, M, k0 + d * 4 * GK, kfin, lane, a[d]);
        load_block<T, B_KCONT, WIDE>(B, ldb, n_tile, N, k0 + d * 4 * GK, kfin, lane, b[d]);
      }
#pragma unroll
      for (int d = 0; d < DEPTH; ++d)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[d][s], b[d][s], acc, 0, 0, 0);
    }
    __shared__ f32x4 sums[4][64];
    sums[wave][lane] = acc;
    __syncthreads();
    // one output per thread: wavefront w takes row 4 (l/16) + w of column l%16
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) v += sums[w][lane][wave];
    store(m_tile + row4 + wave, n_tile + col, v);
  } else {
    const int m0 = m_tile + (wave >> 1) * 16 * F, n0 = n_tile + (wave & 1) * 16 * F;
    f32x4 acc[F][F];
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    float a[2][F][4], b[2][F][4];
    auto load = [&](int buf, int k0) {
#pragma unroll
      for (int i = 0; i < F; ++i) {
        load_block<T, A_KCONT, WIDE>(A, lda, m0 + i * 16, M, k0, kfin, lane, a[buf][i]);
        load_block<T, B_KCONT, WIDE>(B, ldb, n0 + i * 16, N, k0, kfin, lane, b[buf][i]);
      }
    };
    auto multiply = [&](int buf) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < F; ++i)
#pragma unroll
          for (int j = 0; j < F; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[buf][i][s], b[buf][j][s], acc[i][j], 0, 0, 0);
    };
    if (kbeg < kfin) {
      load(0, kbeg);                 // (a step past the k range loads its last k and counts as zero)
      for (int k0 = kbeg; k0 < kfin; k0 += 2 * GK) {
        load(1, k0 + GK);
        multiply(0);
        load(0, k0 + 2 * GK);
        multiply(1);
      }
    }
#pragma unroll
    for (int i = 0; i < F; ++i)
#pragma unroll
      for (int j = 0; j < F; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) store(m0 + i * 16 + row4 + e, n0 + j * 16 + col, acc[i][j][e]);
  }
}

template <typename T, int LAYOUT>
__global__ void finish_kernel(const float* __restrict__ partial, int splits, int M, int N,
                              void* __restrict__ Cv, int ldc, const T* __restrict__ bias,
                              const T* __restrict__ residual, int out_fp32) {
  const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (long)M * N) return;
  const int gm = (int)(i / N), gn = (int)(i % N);
  float v = 0.f;
  for (int z = 0; z < splits; ++z) v += partial[(size_t)z * M * N + i];
  const size_t idx = (size_t)gm * ldc + gn;
  if (LAYOUT == GEMM_TN) { ((float*)Cv)[idx] += v; return; }
  if (bias) v += Elt<T>::to_f(bias[gn]);
  if (residual) v += Elt<T>::to_f(residual[idx]);
  if (out_fp32) ((float*)Cv)[idx] = v;
  else ((T*)Cv)[idx] = Elt<T>::from_f(v);
}

int generic_splits(int M, int N, int K) {
  const long tiles = (long)cdiv(M, GT) * cdiv(N, GT);
  if (tiles >= 128 || K < 1024) return 1;
  int s = (int)(512 / tiles);
  const int by_k = K / 128;
  if (s > by_k) s = by_k;
  if (s > 64) s = 64;
  return s < 1 ? 1 : s;
}

// Blocks per wavefront edge: the largest tile that still gives every CU a workgroup (a wavefront of
// F x F blocks loads 2F blocks of operands for F^2 of products).
int block_edge(int M, int N) {
  if ((long)cdiv(M, 128) * cdiv(N, 128) >= NUM_CU) return 4;
  return (long)cdiv(M, 64) * cdiv(N, 64) >= NUM_CU ? 2 : 1;
}

bool aligned_rows(const void* p, int ld, size_t es) { return reinterpret_cast<uintptr_t>(p) % (4 * es) == 0 && ld % 4 == 0; }

template <typename T, int LAYOUT, int F>
void launch_kernel(bool wide, int M, int N, int K, const T* A, int lda, const T* B, int ldb, void* C, int ldc,
                   const GemmEpilogue& epi, int per, float* partial, int z, const GemmGroups& g, hipStream_t st) {
  constexpr int TILE = F == 1 ? 16 : 32 * F;
  auto kern = wide ? gemm_generic_kernel<T, LAYOUT, F, true> : gemm_generic_kernel<T, LAYOUT, F, false>;
  hipLaunchKernelGGL(kern, dim3(cdiv(N, TILE), cdiv(M, TILE), z), dim3(256), 0, st, M, N, K, A, lda, B, ldb, C, ldc,
                     (const T*)epi.bias, (const T*)epi.residual, epi.out_fp32, per, partial, g);
}

template <typename T>
void launch_layout(int layout, int M, int N, int K, const T* A, int lda, const T* B, int ldb, void* C, int ldc,
                   const GemmEpilogue& epi, int per, float* partial, int z, const GemmGroups& g, hipStream_t st) {
  const int f = block_edge(M, N);
  // every operand whose k is contiguous can be read four values at a time
  const bool wide = K % 4 == 0 && (layout == GEMM_TN || aligned_rows(A, lda, sizeof(T))) &&
                    (layout != GEMM_NT || aligned_rows(B, ldb, sizeof(T))) && g.b_stride % 4 == 0;
#define BM_F(LAY)                                                                                          \
  do {                                                                                                     \
    if (f == 1) launch_kernel<T, LAY, 1>(wide, M, N, K, A, lda, B, ldb, C, ldc, epi, per, partial, z, g, st);      \
    else if (f == 2) launch_kernel<T, LAY, 2>(wide, M, N, K, A, lda, B, ldb, C, ldc, epi, per, partial, z, g, st); \
    else launch_kernel<T, LAY, 4>(wide, M, N, K, A, lda, B, ldb, C, ldc, epi, per, partial, z, g, st);             \
  } while (0)
  if (layout == GEMM_NT) BM_F(GEMM_NT);
  else if (layout == GEMM_NN) BM_F(GEMM_NN);
  else BM_F(GEMM_TN);
#undef BM_F
}

template <typename T>
bm_status launch(int layout, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                 void* C, int ldc, const GemmEpilogue& epi, void* scratch, size_t scratch_bytes,
                 hipStream_t st) {
  int splits = generic_splits(M, N, K);
  if ((size_t)splits * M * N * sizeof(float) > scratch_bytes || !scratch) splits = 1;
  const int per = cdiv(cdiv(K, splits), GK) * GK;
  splits = cdiv(K, per);
  float* partial = splits > 1 ? (float*)scratch : nullptr;
  launch_layout<T>(layout, M, N, K, (const T*)A, lda, (const T*)B, ldb, C, ldc, epi, per, partial, splits, GemmGroups{}, st);
  if (partial) {
    const long n = (long)M * N;
#define BM_F(LAY)                                                                               \
  hipLaunchKernelGGL((finish_kernel<T, LAY>), dim3(cdiv(n, 256)), dim3(256), 0, st, partial,    \
                     splits, M, N, C, ldc, (const T*)epi.bias, (const T*)epi.residual, epi.out_fp32)
    if (layout == GEMM_NT) BM_F(GEMM_NT);
    else if (layout == GEMM_NN) BM_F(GEMM_NN);
    else BM_F(GEMM_TN);
#undef BM_F
  }
  BM_CHECK_LAUNCH("gemm_generic");
  return BM_OK;
}

template <typename T>
bm_status launch_grouped(int layout, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                         void* C, int ldc, const GemmGroups& g, hipStream_t st) {
  launch_layout<T>(layout, M, N, K, (const T*)A, lda, (const T*)B, ldb, C, ldc, GemmEpilogue{}, K, nullptr,
                   layout == GEMM_TN ? g.n_groups : 1, g, st);
  BM_CHECK_LAUNCH("gemm_generic_grouped");
  return BM_OK;
}

}  // namespace

bm_status gemm_generic_grouped(int layout, int dtype, int M, int N, int K, const void* A, int lda,
                               const void* B, int ldb, void* C, int ldc, const GemmGroups& g,
                               hipStream_t st) {
  if (M == 0 || N == 0) return BM_OK;
  GemmGroups gg = g;
  if (layout == GEMM_TN) gg.tile_group = nullptr; else gg.group_rows = nullptr;
  if (dtype == BM_DTYPE_BF16) return launch_grouped<bf16_t>(layout, M, N, K, A, lda, B, ldb, C, ldc, gg, st);
  return launch_grouped<float>(layout, M, N, K, A, lda, B, ldb, C, ldc, gg, st);
}

size_t gemm_generic_scratch_bytes(int M, int N, int K) {
  const int s = generic_splits(M, N, K);
  return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

bm_status gemm_generic(int layout, int dtype, int M, int N, int K, const void* A, int lda,
                       const void* B, int ldb, void* C, int ldc, const GemmEpilogue& epi,
                       void* scratch, size_t scratch_bytes, hipStream_t st) {
  if (M == 0 || N == 0) return BM_OK;
  if (dtype == BM_DTYPE_BF16)
    return launch<bf16_t>(layout, M, N, K, A, lda, B, ldb, C, ldc, epi, scratch, scratch_bytes, st);
  return launch<float>(layout, M, N, K, A, lda, B, ldb, C, ldc, epi, scratch, scratch_bytes, st);
}

}  // namespace bm
