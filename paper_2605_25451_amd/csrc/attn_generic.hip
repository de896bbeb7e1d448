// Variable-length attention with plain fp32 arithmetic: P neighbouring lanes share one
// query row (forward, dq) or one key row (dk, dv) and take every P-th row of the streamed tile,
// which is staged in LDS; their sums meet in lane shuffles at the end.  It serves the fp32 check
// path and head sizes the MFMA kernels do not take.  No atomics: each output element has one owner.
// Bound by the chain of one lane's rows, not by arithmetic or memory: P = 8 against P = 1, fp32 on
// two images of 16 and 24 tokens (4 heads of 16) forward 17.8 -> 9.4 us, dq 12.7 -> 6.3, dk/dv 12.9 -> 7.2.
//
//   forward : o = softmax(q k^T / sqrt(dh) + mask) v,  lse = log sum exp (scaled scores)
//   backward: p = exp(s - lse), dv = p^T do, dp = do v^T, ds = p * (dp - delta),
//             dq = ds k / sqrt(dh), dk = ds^T q / sqrt(dh), delta = rowsum(do * o)
#include "common.h"

#include <type_traits>

namespace bm {

namespace {

constexpr int NT = 128;   // threads per workgroup: NT / P rows
constexpr int BT = 32;    // rows of the streamed tile
// (Functions that several kernels share are always inlined: left as a call, dq with eight lanes at head sizes 32 and 64 held
// 270 registers instead of 150 and moved rows through the stack.  bf16, 16 heads of 32, 997 rows, backward: before they were shared
// 287 us, with the call 325, inlined 169.)

// LDS row stride: the P lanes of a row read P rows of the tile at once (P = 1: all lanes one row)
template <int DH, int P> constexpr int tile_ld() { return P > 1 ? DH + 4 : DH; }

template <int P> __device__ inline float lanes_sum(float v) {
#pragma unroll
  for (int off = 1; off < P; off <<= 1) v += __shfl_xor(v, off, 64);
  return v;
}
template <int P> __device__ inline float lanes_max(float v) {
#pragma unroll
  for (int off = 1; off < P; off <<= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  return v;
}

// BT rows of two matrices from row r0 of `rows` (>= 1) into LDS, `scale` on the first; rows past the last one are zeros.  The
// loads carry no condition (their rows are clamped), so that several are in flight: with a branch around every
// load, here and for a lane's own row, each waited for the one before it.  us, forward / backward: 300 rows, 4 heads of 16, 22 /
// 25 -> 15 / 21; 16 heads of 64 70 / 156 -> 43 / 93; 5 x 200 rows, 8 heads of 128 335 / 803 -> 156 / 373; 4 x 1024 rows, 4 heads of 32,
// 183 / 542 -> 84 / 279.  More than four pairs at once cost registers: all 18 of head size 72 left the forward one wavefront
// per SIMD, and it was slower than with the branches (16 x 1024 rows 923 -> 1045); by sixes 768, 5 x 200 rows of 8 heads 74 -> 40 / 326 -> 190.
template <int DH, int LD, typename T>
__device__ inline void load_tiles(const T* __restrict__ a, int lda, const T* __restrict__ b, int ldb, int r0, int rows, float scale,
                                  float (*A)[LD], float (*B)[LD]) {
  constexpr int N = BT * DH / NT, U = N == 8 ? 8 : N % 4 == 0 ? 4 : N % 6 == 0 ? 6 : N;
  static_assert(BT * DH % NT == 0, "whole trips");
#pragma unroll 1
  for (int it = 0; it < N; it += U) {
    float x[U], y[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = (it + u) * NT + threadIdx.x, r = min(r0 + idx / DH, rows - 1);
      x[u] = Elt<T>::to_f(a[(size_t)r * lda + idx % DH]);
      y[u] = Elt<T>::to_f(b[(size_t)r * ldb + idx % DH]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = (it + u) * NT + threadIdx.x, r = idx / DH;
      A[r][idx % DH] = r0 + r < rows ? x[u] * scale : 0.f;
      B[r][idx % DH] = r0 + r < rows ? y[u] : 0.f;
    }
  }
}

template <typename T, int DH, bool CAUSAL, int P>
__global__ __launch_bounds__(NT) void attn_fwd_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int ld, int ldk,
    const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk, T* __restrict__ o, int ldo,
    float* __restrict__ lse, int Ttot, int group, float scale) {
  constexpr int BQ = NT / P;
  __shared__ float Ks[BT][tile_ld<DH, P>()];
  __shared__ float Vs[BT][tile_ld<DH, P>()];
  const int s = blockIdx.y, hq = blockIdx.z, hk = hq / group;
  const int lo = cu[s], L = cu[s + 1] - lo;
  const int lok = cuk[s], Lk = cuk[s + 1] - lok;     // keys/values may be packed on their own
  const int q0 = blockIdx.x * BQ;
  if (q0 >= L) return;
  const int part = threadIdx.x % P;
  const int qi = q0 + threadIdx.x / P;
  const bool active = qi < L;
  float qr[DH], acc[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) {
    qr[c] = Elt<T>::to_f(q[(size_t)(lo + min(qi, L - 1)) * ld + hq * DH + c]) * scale;
    acc[c] = 0.f;
  }
  float m = -INFINITY, l = 0.f;
  const int kend = CAUSAL ? min(Lk, q0 + BQ) : Lk;
  for (int k0 = 0; k0 < kend; k0 += BT) {
    load_tiles<DH>(k + (size_t)lok * ldk + hk * DH, ldk, v + (size_t)lok * ldk + hk * DH, ldk, k0, Lk, 1.f, Ks, Vs);
    __syncthreads();
    if (active) {
      float sc[BT / P];
      float tmax = -INFINITY;
#pragma unroll
      for (int jj = 0; jj < BT / P; ++jj) {
        const int j = jj * P + part, kj = k0 + j;
        float d = 0.f;
#pragma unroll
        for (int c = 0; c < DH; ++c) d = fmaf(qr[c], Ks[j][c], d);
        bool ok = kj < Lk && (!CAUSAL || kj <= qi);
        sc[jj] = ok ? d : -INFINITY;
        tmax = sc[jj] > tmax || sc[jj] != sc[jj] ? sc[jj] : tmax;   // keeps NaN, which has to reach the row's sums
      }
      if (tmax != -INFINITY) {
        float mn = fmaxf(m, tmax);
        float corr = expf(m - mn);
        l *= corr;
#pragma unroll
        for (int c = 0; c < DH; ++c) acc[c] *= corr;
#pragma unroll
        for (int jj = 0; jj < BT / P; ++jj) {
          const int j = jj * P + part;
          float p = expf(sc[jj] - mn);   // exp(-inf) = 0 for masked keys
          l += p;
#pragma unroll
          for (int c = 0; c < DH; ++c) acc[c] = fmaf(p, Vs[j][c], acc[c]);
        }
        m = mn;
      }
    }
    __syncthreads();
  }
  if (P > 1) {
    // the lanes of a row bring their sums to the common maximum (a lane that saw no key holds zeros)
    const float mall = lanes_max<P>(m);
    const float corr = m > -INFINITY ? expf(m - mall) : 0.f;
    m = mall;
    l = lanes_sum<P>(l * corr);
#pragma unroll
    for (int c = 0; c < DH; ++c) acc[c] = lanes_sum<P>(acc[c] * corr);
  }
  if (active && part == 0) {
    float inv = l > 0.f ? 1.0f / l : 0.f;       // no visible key in this chunk: o = 0, lse = -inf
#pragma unroll
    for (int c = 0; c < DH; ++c)
      o[(size_t)(lo + qi) * ldo + hq * DH + c] = Elt<T>::from_f(acc[c] * inv);
    lse[(size_t)hq * Ttot + lo + qi] = l > 0.f ? m + logf(l) : -INFINITY;
  }
}

// dq, and on the way delta = rowsum(dO * O) of its rows, which a dk/dv kernel of its own reads: a small step is bound by
// its launches, and delta's was one of 27 (4.2 us on its own).  bx: the row tile, s: the sequence, hq: the head.
template <typename T, int DH, bool CAUSAL, int P>
__device__ __forceinline__ void dq_rows(
    int bx, int s, int hq, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int ld, int ldk,
    const T* __restrict__ o, const T* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    float* __restrict__ delta, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk,
    T* __restrict__ dq, int ldd, int Ttot, int group, float scale) {
  constexpr int BQ = NT / P;
  __shared__ float Ks[BT][tile_ld<DH, P>()];
  __shared__ float Vs[BT][tile_ld<DH, P>()];
  const int hk = hq / group;
  const int lo = cu[s], L = cu[s + 1] - lo;
  const int lok = cuk[s], Lk = cuk[s + 1] - lok;
  const int q0 = bx * BQ;
  if (q0 >= L) return;
  const int part = threadIdx.x % P;
  const int qi = q0 + threadIdx.x / P;
  const bool active = qi < L;
  const int qrow = min(qi, L - 1);
  float qr[DH], dor[DH], acc[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) {
    qr[c] = Elt<T>::to_f(q[(size_t)(lo + qrow) * ld + hq * DH + c]) * scale;
    dor[c] = Elt<T>::to_f(d_o[(size_t)(lo + qrow) * ldo + hq * DH + c]);
    acc[c] = 0.f;
  }
  const float my_lse = lse[(size_t)hq * Ttot + lo + qrow];
  float my_delta = 0.f;
#pragma unroll
  for (int c = 0; c < DH; ++c) my_delta = fmaf(Elt<T>::to_f(o[(size_t)(lo + qrow) * ldo + hq * DH + c]), dor[c], my_delta);
  if (active && part == 0) delta[(size_t)hq * Ttot + lo + qi] = my_delta;
  const int kend = CAUSAL ? min(Lk, q0 + BQ) : Lk;
  for (int k0 = 0; k0 < kend; k0 += BT) {
    load_tiles<DH>(k + (size_t)lok * ldk + hk * DH, ldk, v + (size_t)lok * ldk + hk * DH, ldk, k0, Lk, 1.f, Ks, Vs);
    __syncthreads();
    if (active) {
      for (int j = part; j < BT; j += P) {
        int kj = k0 + j;
        if (kj >= Lk || (CAUSAL && kj > qi)) break;
        float sc = 0.f, dp = 0.f;
#pragma unroll
        for (int c = 0; c < DH; ++c) {
          sc = fmaf(qr[c], Ks[j][c], sc);
          dp = fmaf(dor[c], Vs[j][c], dp);
        }
        float ds = expf(sc - my_lse) * (dp - my_delta);
#pragma unroll
        for (int c = 0; c < DH; ++c) acc[c] = fmaf(ds, Ks[j][c], acc[c]);
      }
    }
    __syncthreads();
  }
  if (P > 1) {
#pragma unroll
    for (int c = 0; c < DH; ++c) acc[c] = lanes_sum<P>(acc[c]);
  }
  if (active && part == 0) {
#pragma unroll
    for (int c = 0; c < DH; ++c)
      dq[(size_t)(lo + qi) * ldd + hq * DH + c] = Elt<T>::from_f(acc[c] * scale);
  }
}

template <typename T, int DH, bool CAUSAL, int P>
__global__ __launch_bounds__(NT) void attn_dq_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int ld, int ldk,
    const T* __restrict__ o, const T* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    float* __restrict__ delta, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk,
    T* __restrict__ dq, int ldd, int Ttot, int group, float scale) {
  dq_rows<T, DH, CAUSAL, P>(blockIdx.x, blockIdx.y, blockIdx.z, q, k, v, ld, ldk, o, d_o, ldo, lse, delta, cu, cuk, dq, ldd,
                            Ttot, group, scale);
}

// P lanes per key row of one kv head; the q heads of the group and the query
// tiles are walked in a fixed order, so dk/dv sums are reproducible.
// OWN_DELTA: delta of the streamed rows from o and dO, by the same sum as in dq_rows, instead of from memory.
template <typename T, int DH, bool CAUSAL, int P, bool OWN_DELTA>
__device__ __forceinline__ void dkdv_rows(
    int bx, int s, int hk, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int ld, int ldk,
    const T* __restrict__ o, const T* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cuq, const int32_t* __restrict__ cuk,
    T* __restrict__ dk, T* __restrict__ dv, int ldd, int Ttot, int group, float scale) {
  // this thread's key row lives in the key/value packing (cuk, ldk); queries, dO, lse and
  // delta (Ttot rows per head) in the queries' packing (cuq, ld)
  constexpr int BQ = NT / P;
  __shared__ float Qs[BT][tile_ld<DH, P>()];
  __shared__ float Ds[BT][tile_ld<DH, P>()];
  __shared__ float Ls[BT], Dl[BT];
  const int lok = cuk[s], Lk = cuk[s + 1] - lok;
  const int lo = cuq[s], L = cuq[s + 1] - lo;
  const int kb = bx * BQ;
  if (kb >= Lk) return;
  const int part = threadIdx.x % P;
  const int kj = kb + threadIdx.x / P;
  const bool active = kj < Lk;
  const int krow = min(kj, Lk - 1);
  float kr[DH], vr[DH], dkr[DH], dvr[DH];
#pragma unroll
  for (int c = 0; c < DH; ++c) {
    kr[c] = Elt<T>::to_f(k[(size_t)(lok + krow) * ldk + hk * DH + c]);
    vr[c] = Elt<T>::to_f(v[(size_t)(lok + krow) * ldk + hk * DH + c]);
    dkr[c] = 0.f; dvr[c] = 0.f;
  }
  const int qstart = CAUSAL ? (kb / BT) * BT : 0;
  for (int g = 0; g < group; ++g) {
    const int hq = hk * group + g;
    for (int q0 = qstart; q0 < L; q0 += BT) {
      load_tiles<DH>(q + (size_t)lo * ld + hq * DH, ld, d_o + (size_t)lo * ldo + hq * DH, ldo, q0, L, scale, Qs, Ds);
      if (threadIdx.x < BT) {
        int qi = q0 + threadIdx.x;
        bool ok = qi < L;
        Ls[threadIdx.x] = ok ? lse[(size_t)hq * Ttot + lo + qi] : 0.f;
        float dl = 0.f;
        if (OWN_DELTA && ok) {
          const size_t row = (size_t)(lo + qi) * ldo + hq * DH;
#pragma unroll
          for (int c = 0; c < DH; ++c) dl = fmaf(Elt<T>::to_f(o[row + c]), Elt<T>::to_f(d_o[row + c]), dl);
        } else if (ok) {
          dl = delta[(size_t)hq * Ttot + lo + qi];
        }
        Dl[threadIdx.x] = dl;
      }
      __syncthreads();
      if (active) {
        for (int i = part; i < BT; i += P) {
          int qi = q0 + i;
          if (qi >= L) break;
          if (CAUSAL && kj > qi) continue;
          float sc = 0.f, dp = 0.f;
#pragma unroll
          for (int c = 0; c < DH; ++c) {
            sc = fmaf(Qs[i][c], kr[c], sc);
            dp = fmaf(Ds[i][c], vr[c], dp);
          }
          float p = expf(sc - Ls[i]);
          float ds = p * (dp - Dl[i]);
#pragma unroll
          for (int c = 0; c < DH; ++c) {
            dvr[c] = fmaf(p, Ds[i][c], dvr[c]);
            dkr[c] = fmaf(ds, Qs[i][c], dkr[c]);   // Qs already carries 1/sqrt(dh)
          }
        }
      }
      __syncthreads();
    }
  }
  if (P > 1) {
#pragma unroll
    for (int c = 0; c < DH; ++c) { dkr[c] = lanes_sum<P>(dkr[c]); dvr[c] = lanes_sum<P>(dvr[c]); }
  }
  if (active && part == 0) {
#pragma unroll
    for (int c = 0; c < DH; ++c) {
      dk[(size_t)(lok + kj) * ldd + hk * DH + c] = Elt<T>::from_f(dkr[c]);
      dv[(size_t)(lok + kj) * ldd + hk * DH + c] = Elt<T>::from_f(dvr[c]);
    }
  }
}

template <typename T, int DH, bool CAUSAL, int P>
__global__ __launch_bounds__(NT) void attn_dkdv_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int ld, int ldk,
    const T* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cuq, const int32_t* __restrict__ cuk,
    T* __restrict__ dk, T* __restrict__ dv, int ldd, int Ttot, int group, float scale) {
  dkdv_rows<T, DH, CAUSAL, P, false>(blockIdx.x, blockIdx.y, blockIdx.z, q, k, v, ld, ldk, (const T*)nullptr, d_o, ldo, lse,
                                     delta, cuq, cuk, dk, dv, ldd, Ttot, group, scale);
}

// Both, where eight lanes share a row on either side (few rows): one launch, dk/dv of the Hkv heads in front (they walk the
// heads of their group) and dq of the Hq heads behind.  fp32 block of 40 tokens 91 -> 83 us, of 1000 107 -> 96.  On more rows the sums of delta
// that every dk/dv tile forms for itself cost more than the launch: two launches -> one, 4 heads of 64, 797 rows ahead, 1597 580 -> 621,
// 3997 2864 -> 3090; 4 heads of 16, 3997 rows 367 -> 410 (causal 415 -> 283); 8 / 1 heads of 64, 708 rows 1235 -> 1419.
template <typename T, int DH, bool CAUSAL>
__global__ __launch_bounds__(NT) void attn_bwd_joint_generic_kernel(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, int ld, int ldk,
    const T* __restrict__ o, const T* __restrict__ d_o, int ldo, const float* __restrict__ lse, float* __restrict__ delta,
    const int32_t* __restrict__ cuq, const int32_t* __restrict__ cuk, T* __restrict__ dq, int ldd, T* __restrict__ dk,
    T* __restrict__ dv, int ldd_kv, int Ttot, int Hkv, int group, float scale) {
  const int z = blockIdx.z;
  if (z < Hkv)
    dkdv_rows<T, DH, CAUSAL, 8, true>(blockIdx.x, blockIdx.y, z, q, k, v, ld, ldk, o, d_o, ldo, lse, nullptr, cuq, cuk, dk, dv,
                                      ldd_kv, Ttot, group, scale);
  else
    dq_rows<T, DH, CAUSAL, 8>(blockIdx.x, blockIdx.y, z - Hkv, q, k, v, ld, ldk, o, d_o, ldo, lse, delta, cuq, cuk, dq, ldd,
                              Ttot, group, scale);
}

// Lanes per row.  One lane walks every row of the other side by itself, so few rows leave the chip
// idle behind long chains; eight lanes per row cost eight times the tile loads.  The line was drawn where every load stood behind a branch
// (16 heads of 64, 2048 rows, forward / backward 463 / 1246 -> 370 / 1458, 4096 rows 473 / 1290 -> 564 / 2914).  With the loads of today eight
// lanes are ahead well beyond it: us, forward / backward, P = 1 -> 8: 4 heads of 16, 1000 rows 198 / 456 -> 40 / 53, 8192 1582 / 3662 ->
// 533 / 1477; 16 heads of 64, 1024 686 / 2060 -> 158 / 838, 2048 1370 / 4101 -> 600 / 3203, 4096 2706 / 8040 -> 2508 / 12769; 8 heads of 128, 1024
// 1876 / 7531 -> 344 / 2386, 2048 3741 / 14945 -> 1340 / 9368, 4096 7476 / 29918 -> 5280 / 37396.  The line has not been moved.
bool eight_lanes(long rows, int heads, int dh) { return rows * heads <= 16384 && rows * heads * dh <= (1L << 20); }
template <typename F>
void with_lanes(long rows, int heads, int dh, F&& launch) {
  if (eight_lanes(rows, heads, dh)) launch(std::integral_constant<int, 8>{});
  else launch(std::integral_constant<int, 1>{});
}

template <typename T, int DH, bool CAUSAL>
bm_status fwd_launch(const AttnArgs& a, void* o, float* lse, hipStream_t st) {
  with_lanes(a.T, a.Hq, DH, [&](auto p) {
    constexpr int P = decltype(p)::value;
    hipLaunchKernelGGL((attn_fwd_generic_kernel<T, DH, CAUSAL, P>), dim3(cdiv(a.max_seqlen, NT / P), a.S, a.Hq), dim3(NT),
                       0, st, (const T*)a.q, (const T*)a.k, (const T*)a.v, a.ld_qkv, a.kv_ld(), a.cu_dev, a.kv_cu_dev(),
                       (T*)o, a.Hq * a.dh, lse, a.T, a.Hq / a.Hkv, 1.0f / sqrtf((float)a.dh));
  });
  BM_CHECK_LAUNCH("attn_fwd_generic");
  return BM_OK;
}

template <typename T, int DH, bool CAUSAL>
bm_status bwd_launch(const AttnArgs& a, const void* o, const void* d_o, const float* lse, void* dq,
                     void* dk, void* dv, int ldd, float* delta, hipStream_t st) {
  const int ldo = a.Hq * a.dh;
  const float scale = 1.0f / sqrtf((float)a.dh);
  if constexpr (DH <= 64)
    if (!a.in_place && a.T > 0 && a.kv_T() > 0 && eight_lanes(a.T, a.Hq, DH) && eight_lanes(a.kv_T(), a.Hkv, DH)) {
      const int longest = a.max_seqlen > a.kv_max_len() ? a.max_seqlen : a.kv_max_len();
      hipLaunchKernelGGL((attn_bwd_joint_generic_kernel<T, DH, CAUSAL>), dim3(cdiv(longest, NT / 8), a.S, a.Hkv + a.Hq), dim3(NT),
                         0, st, (const T*)a.q, (const T*)a.k, (const T*)a.v, a.ld_qkv, a.kv_ld(), (const T*)o, (const T*)d_o,
                         ldo, lse, delta, a.cu_dev, a.kv_cu_dev(), (T*)dq, ldd, (T*)dk, (T*)dv,
                         a.ld_dkv ? a.ld_dkv : ldd, a.T, a.Hkv, a.Hq / a.Hkv, scale);
      BM_CHECK_LAUNCH("attn_bwd_generic");
      return BM_OK;
    }
  if (a.T > 0) {
    with_lanes(a.T, a.Hq, DH, [&](auto p) {
      constexpr int P = decltype(p)::value;
      hipLaunchKernelGGL((attn_dq_generic_kernel<T, DH, CAUSAL, P>), dim3(cdiv(a.max_seqlen, NT / P), a.S, a.Hq),
                         dim3(NT), 0, st, (const T*)a.q, (const T*)a.k, (const T*)a.v, a.ld_qkv, a.kv_ld(),
                         (const T*)o, (const T*)d_o, ldo, lse, delta, a.cu_dev, a.kv_cu_dev(), (T*)dq, ldd, a.T,
                         a.Hq / a.Hkv, scale);
    });
  }
  if (a.kv_T() > 0)
    with_lanes(a.kv_T(), a.Hkv, DH, [&](auto p) {
      constexpr int P = decltype(p)::value;
      hipLaunchKernelGGL((attn_dkdv_generic_kernel<T, DH, CAUSAL, P>), dim3(cdiv(a.kv_max_len(), NT / P), a.S, a.Hkv),
                         dim3(NT), 0, st, (const T*)a.q, (const T*)a.k, (const T*)a.v, a.ld_qkv, a.kv_ld(),
                         (const T*)d_o, ldo, lse, delta, a.cu_dev, a.kv_cu_dev(), (T*)dk, (T*)dv,
                         a.ld_dkv ? a.ld_dkv : ldd, a.T, a.Hq / a.Hkv, scale);
    });
  BM_CHECK_LAUNCH("attn_bwd_generic");
  return BM_OK;
}

#define BM_DH_SWITCH(CALL)                      \
  switch (a.dh) {                               \
    case 8: CALL(8); break;                     \
    case 16: CALL(16); break;                   \
    case 32: CALL(32); break;                   \
    case 64: CALL(64); break;                   \
    case 72: CALL(72); break;                   \
    case 128: CALL(128); break;                 \
    default:                                    \
      set_error("attention: head_dim %d unsupported (8,16,32,64,72,128)", a.dh); \
      return BM_ERR_UNSUPPORTED;                \
  }

}  // namespace

bm_status attention_forward_generic(const AttnArgs& a, void* o, float* lse, hipStream_t st) {
  if (a.T == 0) return BM_OK;
#define BM_CALL(D)                                                                             \
  if (a.dtype == BM_DTYPE_BF16)                                                                \
    return a.causal ? fwd_launch<bf16_t, D, true>(a, o, lse, st) : fwd_launch<bf16_t, D, false>(a, o, lse, st); \
  else                                                                                         \
    return a.causal ? fwd_launch<float, D, true>(a, o, lse, st) : fwd_launch<float, D, false>(a, o, lse, st)
  BM_DH_SWITCH(BM_CALL)
#undef BM_CALL
  return BM_OK;
}

bm_status attention_backward_generic(const AttnArgs& a, const void* o, const void* d_o,
                                     const float* lse, void* dq, void* dk, void* dv, int ldd,
                                     float* delta, hipStream_t st) {
  if (a.T == 0 && a.kv_T() == 0) return BM_OK;
#define BM_CALL(D)                                                                             \
  if (a.dtype == BM_DTYPE_BF16)                                                                \
    return a.causal ? bwd_launch<bf16_t, D, true>(a, o, d_o, lse, dq, dk, dv, ldd, delta, st)  \
                    : bwd_launch<bf16_t, D, false>(a, o, d_o, lse, dq, dk, dv, ldd, delta, st); \
  else                                                                                         \
    return a.causal ? bwd_launch<float, D, true>(a, o, d_o, lse, dq, dk, dv, ldd, delta, st)   \
                    : bwd_launch<float, D, false>(a, o, d_o, lse, dq, dk, dv, ldd, delta, st)
  BM_DH_SWITCH(BM_CALL)
#undef BM_CALL
  return BM_OK;
}

}  // namespace bm
