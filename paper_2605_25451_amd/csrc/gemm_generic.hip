// Shape-agnostic GEMM with fp32 arithmetic.  It is the fp32 check path of
// the block and the cover for shapes the bf16 MFMA kernels do not take (tiny or
// oddly sized problems such as the adaLN conditioning projection).
//
//   NT: C[M,N]  = A[M,K] B[N,K]^T      NN: C[M,N] = A[M,K] B[K,N]
//   TN: C[M,N] += A[K,M]^T B[K,N]      (C fp32, accumulated)
//
// Two kernels.  In gemm_direct_kernel operands go from memory straight into the registers of
// v_mfma_f32_16x16x4_f32: no LDS, no barrier in the loop, and many loads in flight, which is what small products,
// bound by latency, want; every wavefront reads its own rows.  gemm_tiled_kernel stages 64x64 tiles in LDS, so that
// how the rows lie costs little, but pays a memory latency and two barriers per 16 k.  See choose_kernel()
// for the line between them.  Every access of either is clamped into its matrix or left out, and what lies past the
// k range counts as zero.
#include "common.h"

namespace bm {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int NUM_CU = 256;
constexpr int GT = 64;   // tile edge of the tiled kernel, for which the k split is chosen too
constexpr int GK = 16;   // k step (direct kernel: four MFMAs; lane l holds k = 4 (l/16) + s of step s)

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
// four sums meet in LDS.  F = 2: a wavefront owns 2x2 blocks, a workgroup 64x64.
// With k_per_split < K the grid's z index selects a k range and the workgroup stores
// its fp32 partial tile into `partial` [z][M][N]; finish_kernel then sums the ranges
// in order and applies the epilogue (skinny problems: few output tiles, long K).
struct DirectGelu { void* a; const void* up; void* dup; void* act; float* sums; };   // see GemmEpilogue; 16x16 tiles, one k range
template <typename T, int LAYOUT, int F, bool WIDE>
__device__ inline void direct_tile(dim3 at,
    int M, int N, int K, const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
    void* __restrict__ Cv, int ldc, const T* __restrict__ bias, const T* __restrict__ residual,
    int out_fp32, int k_per_split, float* __restrict__ partial, GemmGroups grp, DirectGelu gelu = {}) {
  constexpr int TILE = F == 1 ? 16 : 32 * F;
  constexpr bool A_KCONT = LAYOUT != GEMM_TN, B_KCONT = LAYOUT == GEMM_NT;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m_tile = (int)at.y * TILE, n_tile = (int)at.x * TILE;
  int kbeg = (int)at.z * k_per_split;
  int kfin = min(K, kbeg + k_per_split);
  if (grp.group_rows) {              // grouped weight gradient: the z index is the group
    kbeg = min(grp.group_rows[at.z], K);
    kfin = min(grp.group_rows[at.z + 1], K);
    if (kbeg >= kfin) return;
    Cv = (float*)Cv + (long)at.z * grp.c_stride;
  } else if (grp.tile_group) {       // grouped forward / input gradient: B of this row block's group
    const int g = grp.tile_group[m_tile / MOE_PAD];
    if (g < 0) return;
    B += (long)g * grp.b_stride;
  }
  auto store = [&](int gm, int gn, float v) {
    if (gm >= M || gn >= N) return;
    const size_t idx = (size_t)gm * ldc + gn;
    if (partial) {
      partial[((size_t)at.z * M + gm) * N + gn] = v;
    } else if (LAYOUT == GEMM_TN) {
      ((float*)Cv)[idx] += v;
    } else {
      if (bias) v += Elt<T>::to_f(bias[gn]);
      if (residual) v += Elt<T>::to_f(residual[idx]);
      if (out_fp32) ((float*)Cv)[idx] = v;
      else ((T*)Cv)[idx] = Elt<T>::from_f(v);
      if (LAYOUT == GEMM_NT && F == 1 && gelu.a) ((T*)gelu.a)[idx] = Elt<T>::from_f(gelu_f(Elt<T>::to_f(Elt<T>::from_f(v))));
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
    if (LAYOUT == GEMM_NN && gelu.up) {
      const int gm = m_tile + row4 + wave, gn = n_tile + col;
      float d = 0.f;
      if (gm < M && gn < N) {
        const size_t idx = (size_t)gm * N + gn;
        const float z = Elt<T>::to_f(((const T*)gelu.up)[idx]);
        float cdf, pdf;
        normal_cdf_pdf(z, &cdf, &pdf);
        const T stored = Elt<T>::from_f(v * (cdf + z * pdf));
        ((T*)gelu.dup)[idx] = stored;
        ((T*)gelu.act)[idx] = Elt<T>::from_f(z * cdf);
        d = Elt<T>::to_f(stored);
      }
      if (gelu.sums) {
        d += __shfl_xor(d, 16, WAVE);
        d += __shfl_xor(d, 32, WAVE);
        __syncthreads();
        float* rows4 = reinterpret_cast<float*>(sums);
        if (lane < 16) rows4[wave * 16 + lane] = d;
        __syncthreads();
        if (wave == 0 && lane < 16 && gn < N) {
          const float* s = rows4 + lane;
          gelu.sums[(size_t)at.y * N + gn] = (s[0] + s[16]) + (s[32] + s[48]);
        }
      }
      return;
    }
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

template <typename T, int LAYOUT, int F, bool WIDE>
__global__ __launch_bounds__(256) void gemm_direct_kernel(
    int M, int N, int K, const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
    void* __restrict__ Cv, int ldc, const T* __restrict__ bias, const T* __restrict__ residual,
    int out_fp32, int k_per_split, float* __restrict__ partial, GemmGroups grp, DirectGelu gelu) {
  direct_tile<T, LAYOUT, F, WIDE>(dim3(blockIdx.x, blockIdx.y, blockIdx.z), M, N, K, A, lda, B, ldb, Cv, ldc, bias, residual,
                                  out_fp32, k_per_split, partial, grp, gelu);
}

// An input and a weight gradient of few rows in one grid (16x16 tiles): what either costs alone is a launch (fp32 block
// of 64 columns, three such pairs: 40 tokens 99 -> 87 us, 300 tokens 104 -> 92).
template <typename T, bool WIDE_NN, bool WIDE_TN>
__global__ __launch_bounds__(256) void gemm_direct_joint_kernel(GemmCall nn, GemmCall tn, int nn_wgs) {
  const bool first = (int)blockIdx.x < nn_wgs;
  const int id = first ? blockIdx.x : blockIdx.x - nn_wgs, across = (first ? nn.N + 15 : tn.N + 15) / 16;
  const dim3 at(id % across, id / across, 0);
  if (first)
    direct_tile<T, GEMM_NN, 1, WIDE_NN>(at, nn.M, nn.N, nn.K, (const T*)nn.A, nn.lda, (const T*)nn.B, nn.ldb, nn.C, nn.ldc,
                                        (const T*)nullptr, (const T*)nullptr, 0, nn.K, nullptr, GemmGroups{});
  else
    direct_tile<T, GEMM_TN, 1, WIDE_TN>(at, tn.M, tn.N, tn.K, (const T*)tn.A, tn.lda, (const T*)tn.B, tn.ldb, tn.C, tn.ldc,
                                        (const T*)nullptr, (const T*)nullptr, 0, tn.K, nullptr, GemmGroups{});
}

// 64x64 output tile per workgroup, 16-deep k slices staged in LDS, a 4x4 register tile per thread.  Every
// access is bounds-checked.  k ranges as above.
template <typename T, int LAYOUT>
__global__ __launch_bounds__(256) void gemm_tiled_kernel(
    int M, int N, int K, const T* __restrict__ A, int lda, const T* __restrict__ B, int ldb,
    void* __restrict__ Cv, int ldc, const T* __restrict__ bias, const T* __restrict__ residual,
    int out_fp32, int k_per_split, float* __restrict__ partial, GemmGroups grp, DirectGelu) {
  __shared__ float As[GK][GT + 4];
  __shared__ float Bs[GK][GT + 4];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * GT, n0 = blockIdx.x * GT;
  int kbeg = blockIdx.z * k_per_split;
  int kfin = min(K, kbeg + k_per_split);
  if (grp.group_rows) {              // grouped weight gradient: blockIdx.z is the group
    kbeg = min(grp.group_rows[blockIdx.z], K);
    kfin = min(grp.group_rows[blockIdx.z + 1], K);
    if (kbeg >= kfin) return;
    Cv = (float*)Cv + (long)blockIdx.z * grp.c_stride;
  } else if (grp.tile_group) {       // grouped forward / input gradient: B of this row block's group
    const int g = grp.tile_group[m0 / MOE_PAD];
    if (g < 0) return;
    B += (long)g * grp.b_stride;
  }
  const int ty = tid >> 4, tx = tid & 15;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;

  for (int k0 = kbeg; k0 < kfin; k0 += GK) {
    // A slice -> As[k][m]
    if (LAYOUT == GEMM_TN) {
      int k = tid >> 4, m = (tid & 15) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int gm = m0 + m + e, gk = k0 + k;
        As[k][m + e] = (gm < M && gk < kfin) ? Elt<T>::to_f(A[(size_t)gk * lda + gm]) : 0.f;
      }
    } else {
      int m = tid >> 2, k = (tid & 3) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int gm = m0 + m, gk = k0 + k + e;
        As[k + e][m] = (gm < M && gk < kfin) ? Elt<T>::to_f(A[(size_t)gm * lda + gk]) : 0.f;
      }
    }
    // B slice -> Bs[k][n]
    if (LAYOUT == GEMM_NT) {
      int n = tid >> 2, k = (tid & 3) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int gn = n0 + n, gk = k0 + k + e;
        Bs[k + e][n] = (gn < N && gk < kfin) ? Elt<T>::to_f(B[(size_t)gn * ldb + gk]) : 0.f;
      }
    } else {
      int k = tid >> 4, n = (tid & 15) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int gn = n0 + n + e, gk = k0 + k;
        Bs[k][n + e] = (gn < N && gk < kfin) ? Elt<T>::to_f(B[(size_t)gk * ldb + gn]) : 0.f;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < GK; ++k) {
      float a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[k][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[k][tx * 4 + j];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], b[j], acc[i][j]);
    }
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int gm = m0 + ty * 4 + i;
    if (gm >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int gn = n0 + tx * 4 + j;
      if (gn >= N) continue;
      size_t idx = (size_t)gm * ldc + gn;
      float v = acc[i][j];
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
    }
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

bool aligned_rows(const void* p, int ld, size_t es) { return reinterpret_cast<uintptr_t>(p) % (4 * es) == 0 && ld % 4 == 0; }

// Which kernel: 0 tiled, else F of the direct one.
//  - Few 64x64 tiles x k ranges per CU (`load`) are bound by the chain of k steps: one 16x16 tile per workgroup, whose
//    wavefronts share the k range.  Later its loads (64 values per 16 products) cost more than the chain:
//    2x2 blocks.
//  - Where k is contiguous (NT, NN), one value at a time or four bf16 values leave most of every 64-byte segment that
//    is requested unused, and a short contraction is nothing but those requests: the tiled kernel, from about a
//    workgroup per CU on (NN: one of its operands is read along its rows).  The same goes for bf16 weight gradients
//    of less than a k step (12288x4096 over 3 rows 147 / 318 / 165 us).
// us, tiled / direct with 16x16 / with 2x2 blocks.  fp32: NT 40x64x256 27.5 / 8.2 / -, 1028^3 135 / 65 / 55, 2052^3 421 / 468 / 272,
// TN 2052^3 353 / 590 / 275; odd rows, NT 1540^3 271 / 557 / 362, 1000x256x1024 31 / 75 / 29.  bf16: NT 2052^3 384 / 922 / 585, NN 343 /
// 565 / 373, TN 302 / 454 / 313.  Over 4226 shapes of both types, 24 to 6000 rows and columns and K from 1 to 4000: 30 % less time
// than the tiled kernel alone (geometric mean), 2.4 % more than the best of the three.
int choose_kernel(int layout, int M, int N, int K, int z, bool bf16, bool wide) {
  const double load = (double)cdiv(M, GT) * cdiv(N, GT) * z / NUM_CU;
  if (load < (wide || layout == GEMM_TN ? 0.75 : 0.5)) return 1;
  if (layout == GEMM_TN) return bf16 && K < 16 ? 0 : 2;
  if (wide && !bf16) return 2;
  if (wide && K < 80) return 0;
  return load < (layout == GEMM_NT ? 1.0 : wide ? 2.0 : 3.0) ? 2 : 0;
}

template <typename T, int LAYOUT>
void launch_kernel(int which, bool wide, int M, int N, int K, const T* A, int lda, const T* B, int ldb, void* C, int ldc,
                   const GemmEpilogue& epi, int per, float* partial, int z, const GemmGroups& g, hipStream_t st) {
  const int tile = which == 1 ? 16 : 64;
  auto kern = which == 0 ? gemm_tiled_kernel<T, LAYOUT>
            : which == 1 ? (wide ? gemm_direct_kernel<T, LAYOUT, 1, true> : gemm_direct_kernel<T, LAYOUT, 1, false>)
                         : (wide ? gemm_direct_kernel<T, LAYOUT, 2, true> : gemm_direct_kernel<T, LAYOUT, 2, false>);
  hipLaunchKernelGGL(kern, dim3(cdiv(N, tile), cdiv(M, tile), z), dim3(256), 0, st, M, N, K, A, lda, B, ldb, C, ldc,
                     (const T*)epi.bias, (const T*)epi.residual, epi.out_fp32, per, partial, g,
                     DirectGelu{epi.gelu_a, epi.gelu_up, epi.gelu_dup, epi.gelu_act, epi.gelu_sums});
}

template <typename T>
void launch_layout(int layout, int M, int N, int K, const T* A, int lda, const T* B, int ldb, void* C, int ldc,
                   const GemmEpilogue& epi, int per, float* partial, int z, const GemmGroups& g, hipStream_t st) {
  // every operand whose k is contiguous can be read four values at a time
  const bool wide = K % 4 == 0 && (layout == GEMM_TN || aligned_rows(A, lda, sizeof(T))) &&
                    (layout != GEMM_NT || aligned_rows(B, ldb, sizeof(T))) && g.b_stride % 4 == 0;
  const int which = choose_kernel(layout, M, N, K, z, sizeof(T) == 2, wide);
  if (layout == GEMM_NT) launch_kernel<T, GEMM_NT>(which, wide, M, N, K, A, lda, B, ldb, C, ldc, epi, per, partial, z, g, st);
  else if (layout == GEMM_NN) launch_kernel<T, GEMM_NN>(which, wide, M, N, K, A, lda, B, ldb, C, ldc, epi, per, partial, z, g, st);
  else launch_kernel<T, GEMM_TN>(which, wide, M, N, K, A, lda, B, ldb, C, ldc, epi, per, partial, z, g, st);
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

// GELU in the epilogue of 16x16 tiles with one k range, contiguous aligned rows: at these sizes a launch costs as much as a product
// (fp32 block of 64 columns, two launches of 17 fewer: 70 -> 64 us of kernels at 40 tokens; a pass of 300 tokens 88 -> 84 us, 1000 tokens
// 107 -> 102, 2000 tokens 141 -> 136; bf16 tiles of 128x128 gain nothing: 300 to 1000 rows of 1024 columns within 0.5 %).
bool gemm_fuses_gelu(int layout, int dtype, int M, int N, int K) {
  return dtype == BM_DTYPE_FP32 && layout != GEMM_TN && generic_splits(M, N, K) == 1 && K % 4 == 0 &&
         choose_kernel(layout, M, N, K, 1, false, true) == 1;
}

static bool wide_nn(const GemmCall& g) { return g.K % 4 == 0 && aligned_rows(g.A, g.lda, sizeof(float)); }

// both products as the separate launches would run them: 16x16 tiles, one k range
bool gemm_generic_nn_tn_shares(int dtype, const GemmCall& nn, const GemmCall& tn) {
  return dtype == BM_DTYPE_FP32 && generic_splits(nn.M, nn.N, nn.K) == 1 && generic_splits(tn.M, tn.N, tn.K) == 1 &&
         choose_kernel(GEMM_NN, nn.M, nn.N, nn.K, 1, false, wide_nn(nn)) == 1 &&
         choose_kernel(GEMM_TN, tn.M, tn.N, tn.K, 1, false, tn.K % 4 == 0) == 1;
}

bool gemm_generic_nn_tn(int dtype, const GemmCall& nn, const GemmCall& tn, hipStream_t st, bm_status* rc) {
  if (!gemm_generic_nn_tn_shares(dtype, nn, tn)) return false;
  const bool wide0 = wide_nn(nn), wide1 = tn.K % 4 == 0;
  ProfScope prof(PROF_GEMM_NN, 2.0 * nn.M * nn.N * nn.K + 2.0 * tn.M * tn.N * tn.K, st);       // the class of the first
  const int wgs0 = cdiv(nn.M, 16) * cdiv(nn.N, 16), wgs1 = cdiv(tn.M, 16) * cdiv(tn.N, 16);
  auto kern = wide0 ? (wide1 ? gemm_direct_joint_kernel<float, true, true> : gemm_direct_joint_kernel<float, true, false>)
                    : (wide1 ? gemm_direct_joint_kernel<float, false, true> : gemm_direct_joint_kernel<float, false, false>);
  hipLaunchKernelGGL(kern, dim3(wgs0 + wgs1), dim3(256), 0, st, nn, tn, wgs0);
  const hipError_t e = hipGetLastError();
  *rc = e == hipSuccess ? BM_OK : hip_fail(e, "gemm_direct_joint");
  return true;
}

size_t gemm_generic_scratch_bytes(int M, int N, int K) {
  const int s = generic_splits(M, N, K);
  return s > 1 ? (size_t)s * M * N * sizeof(float) : 0;
}

bm_status gemm_generic(int layout, int dtype, int M, int N, int K, const void* A, int lda,
                       const void* B, int ldb, void* C, int ldc, const GemmEpilogue& epi,
                       void* scratch, size_t scratch_bytes, hipStream_t st) {
  if (M == 0 || N == 0) return BM_OK;
  if ((epi.gelu_a || epi.gelu_up) && !(gemm_fuses_gelu(layout, dtype, M, N, K) && ldc == N)) {
    set_error("gemm: no GELU in the epilogue of this product");
    return BM_ERR_UNSUPPORTED;
  }
  if (dtype == BM_DTYPE_BF16)
    return launch<bf16_t>(layout, M, N, K, A, lda, B, ldb, C, ldc, epi, scratch, scratch_bytes, st);
  return launch<float>(layout, M, N, K, A, lda, B, ldb, C, ldc, epi, scratch, scratch_bytes, st);
}

}  // namespace bm
