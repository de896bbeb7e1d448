// bf16 GEMM on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16), fp32 accumulation: the choice of tile and
// k split, and the kernel of 128x128 tiles (the other tiles: gemm_alt.hip).
//
//   NT: C[M,N]  = A[M,K] B[N,K]^T (+bias)(+residual)   linear forward
//   NN: C[M,N]  = A[M,K] B[K,N]                        input gradient
//   TN: C[M,N] += A[K,M]^T B[K,N]     (C fp32)         weight gradient
//
// The 128x128 kernel serves outputs of few tiles, two workgroups per CU: four wavefronts of 64x64, K in
// slices of BK=64, both operand slices staged in LDS (two buffers: the next slice is fetched from
// memory into registers while the current one feeds the MFMAs, one barrier per
// slice).  An operand whose K index is contiguous in memory is kept as
// [row][k] with its 16-byte chunks XOR-swizzled by the row, and fragments are
// read with ds_read_b128.  An operand whose K index is the slow one (B of NN,
// both operands of TN) is kept as [k][row] and fragments are read with the
// LDS transpose read (ds_read_b64_tr_b16), so no transposed copy is ever made.
// Workgroup ids are remapped so that the workgroups of one XCD (they share an
// L2) cover a compact block of tiles.  A split k range leaves fp32 partial
// tiles that a second kernel sums in a fixed order: no floating-point atomics.
#include "gemm_tile.h"

#include <atomic>

namespace bm {

namespace {

// ---- LDS layouts ---------------------------------------------------------
// k-contiguous operand: [rows][KCH chunks]; chunk c of row r sits at c ^ ((r>>1)&7).
__device__ inline int kc_offset(int row, int c) {          // in bf16 elements
  return row * BK + ((c ^ ((row >> 1) & (KCH - 1))) << 3);
}
// transposed operand: [BK k-rows][R/8 chunks]; chunk c of k-row k sits at
// c ^ ((k&3)<<2) ^ (((k>>3)&1)<<1): a transpose read touches 4 consecutive k-rows x 32 bytes
// per 16 lanes; the first term puts the 4 k-rows into different 64-byte bank windows, the
// second moves the lane group that reads 8 k-rows further on into the other half of each.
template <int R>
__device__ inline int tr_offset(int k, int c) {             // in bf16 elements
  const int pos = c ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1);
  return k * R + (pos << 3);
}

// 16(row) x 32(k) fragments of the v_mfma_f32_16x16x32_bf16 operands: lane l holds row
// row0 + l%16 and k = k0 + (l/16)*8 .. +7.
__device__ inline bf16x8 kc_fragment16(const bf16_t* lds, int row0, int ks32, int lane) {
  const int row = row0 + (lane & 15);
  const int c = ks32 * 4 + (lane >> 4);
  return *reinterpret_cast<const bf16x8*>(lds + kc_offset(row, c));
}

template <int R>
__device__ inline bf16x8 tr_fragment16(const bf16_t* lds, int row0, int k0, int lane) {
  // operand stored [k][row]: the 16 lanes of group gi read a 4(k) x 16(row) block, 8 bytes each, and
  // the transpose read hands lane s row row0 + s with 4 consecutive k; two reads give 8 k
  const int gi = lane >> 4, s = lane & 15;
  const int r = row0 + (s & 3) * 4;
  const int k = k0 + gi * 8 + (s >> 2);
  const int c = r >> 3, within = r & 7;
  const bf16_t* p0 = lds + tr_offset<R>(k, c) + within;
  const bf16_t* p1 = lds + tr_offset<R>(k + 4, c) + within;
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p1);
  union { struct { s16x4 a, b; } s; bf16x8 v; } u;
  u.s.a = lo; u.s.b = hi;
  return u.v;
}

// ---- global -> registers -> LDS staging -----------------------------------
// Each thread moves CH = (R*BK/8)/NT chunks of 16 bytes per slice and operand.
// A chunk's position inside a slice never changes, so its global offset (relative
// to a wave-uniform slice base pointer that the caller advances) and its LDS offset
// are computed once; per slice a chunk costs one load and one LDS store.
template <int R, int NT, bool TR, bool KTAIL>
struct Stage {
  static constexpr int CH = (R * BK / 8) / NT;
  static constexpr int PARTS = BK / 32;          // one part per k-step (k = 32) of the MFMA loop
  static constexpr int PER = CH / PARTS;
  static_assert(CH % PARTS == 0, "tile does not split evenly over the k-steps");
  u32x4 v[CH];
  uint32_t goff[CH];    // byte offset from the slice base pointer
  unsigned live = 0u;   // KTAIL: bit i = chunk i lies inside the k range (else stored as zeros)
  // LDS byte offset of chunk i = soff + i * SSTRIDE: from one chunk of a thread to the next
  // the row (k-contiguous layout) or the k-row (transposed layout) advances by a fixed count that
  // leaves the XOR swizzle alone
  static constexpr int IROWS = TR ? NT / (R / 8) : NT / KCH;      // rows (k-rows) between chunks i and i+1
  static constexpr int SSTRIDE = IROWS * (TR ? R : BK) * 2;
  static_assert(IROWS % 16 == 0, "the chunk stride would move the swizzle");
  uint32_t soff;

  // k index of chunk i inside a slice
  __device__ static inline int chunk_k(int i, int tid) {
    const int id = tid + i * NT;
    return TR ? id / (R / 8) : (id % KCH) * 8;
  }
  // rows_left: how many rows of the R dimension are valid from this tile's first row on
  // half > 0 (k-contiguous operand only): the tile's rows are gathered from two row ranges F rows
  // apart -- within every run of 2*half tile rows, the first half come from row0.. and the second
  // half from F + row0.. (the gate and the up half of a SwiGLU weight); offsets are then relative
  // to the matrix's first row
  __device__ inline void init(int ld, int rows_left, int tid, int half = 0, int F = 0, int row0 = 0) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int id = tid + i * NT;
      if (!TR && half > 0) {
        const int r = id / KCH;
        const int row = (r / half & 1) * F + row0 + (r / (2 * half)) * half + r % half;
        goff[i] = ((uint32_t)row * (uint32_t)ld + (uint32_t)(id % KCH) * 8u) * 2u;
        continue;
      }
      if (TR) {            // memory [k][row]: chunk = 8 consecutive rows
        int row = (id % (R / 8)) * 8;
        if (row >= rows_left) row = 0;
        goff[i] = ((uint32_t)(id / (R / 8)) * (uint32_t)ld + (uint32_t)row) * 2u;
      } else {             // memory [row][k]: chunk = 8 consecutive k
        int row = id / KCH;
        if (row >= rows_left) row = rows_left - 1;
        goff[i] = ((uint32_t)row * (uint32_t)ld + (uint32_t)(id % KCH) * 8u) * 2u;
      }
    }
    soff = (uint32_t)(TR ? tr_offset<R>(tid / (R / 8), tid % (R / 8)) : kc_offset(tid / KCH, tid % KCH)) * 2u;
  }

  // base: this tile's first row at the slice's first k (wave-uniform); k_left = valid k from there
  __device__ inline void load_one(int i, const bf16_t* __restrict__ base, int ld, int k_left, int tid) {
    uint32_t o = goff[i];
    if (KTAIL) {
      // keep the address valid and remember to store zeros instead
      const int kk = chunk_k(i, tid);
      const bool in = kk < k_left;
      live = (live & ~(1u << i)) | ((in ? 1u : 0u) << i);
      if (!in) o -= (TR ? (uint32_t)(kk - (k_left - 1)) * (uint32_t)ld : (uint32_t)(kk - (k_left - 8))) * 2u;
    }
    // the empty asm keeps the widening of the 32-bit offset next to the load, where the instruction
    // selector can fold it into the scalar-base + 32-bit-offset address form (hoisted out of the loop
    // it becomes a 64-bit register pair and a 64-bit add per load)
    asm volatile("" : "+v"(o));
    v[i] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(base) + o);
  }

  __device__ inline void store_one(int i, bf16_t* lds) const {
    u32x4 val = v[i];
    if (KTAIL && !((live >> i) & 1u)) val = u32x4{0u, 0u, 0u, 0u};
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(lds) + soff + i * SSTRIDE) = val;
  }

  __device__ inline void load(const bf16_t* __restrict__ base, int ld, int k_left, int tid) {
#pragma unroll
    for (int i = 0; i < CH; ++i) load_one(i, base, ld, k_left, tid);
  }
  __device__ inline void store(bf16_t* lds) const {
#pragma unroll
    for (int i = 0; i < CH; ++i) store_one(i, lds);
  }
};

// one workgroup's tile: pid among the workgroups of its product
template <bool A_TR, bool B_TR, int EPI, bool KTAIL>
__device__ inline void small_tile(GemmParams p, int pid) {
  constexpr int BM = 128, BN = 128, WM = 2, WN = 2, NT = WM * WN * 64;
  constexpr int TM = BM / WM, TN_ = BN / WN;       // wave tile
  constexpr int FM = TM / 16, FN = TN_ / 16;       // 16x16 blocks per wave
  extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
  bf16_t* smem = reinterpret_cast<bf16_t*>(smem_raw);
  constexpr int A_TILE = BM * BK, B_TILE = BN * BK;      // elements; buffers: A0 A1 B0 B1

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;

  const TileJob job = locate_tile<BM, BN>(p, pid);
  if (job.kbeg >= job.kend) return;
  const int m0 = job.m0, n0 = job.n0, kbeg = job.kbeg, kend = job.kend;

  f32x4 acc[FM][FN];        // first written by the first k-step of the first slice

  // Software pipeline, two slices deep: the registers of `sa`/`sb` always hold the
  // slice after the one being multiplied.  During k-step ks of slice j, part ks of
  // slice j+1 (fetched one whole slice ago) is written to the free LDS buffer and
  // the same registers are re-armed with part ks of slice j+2, so HBM/L2 latency is
  // covered by a full slice of MFMAs and memory instructions are spread between them.
  Stage<BM, NT, A_TR, KTAIL> sa;
  Stage<BN, NT, B_TR, KTAIL> sb;
  sa.init(p.lda, p.M - m0, tid);
  constexpr bool swf = EPI == EPI_SWIGLU_FWD;            // SwiGLU forward: N = 2F, a tile covers BN/2 columns of a
  if (swf) sb.init(p.ldb, BN, tid, TN_ / 2, p.N / 2, job.tn * (BN / 2));
  else sb.init(p.ldb, p.N - n0, tid);
  // slice base pointers (wave-uniform): first row of the tile at k = kbeg
  const bf16_t* a_base = A_TR ? job.A + (size_t)kbeg * p.lda + m0 : job.A + (size_t)m0 * p.lda + kbeg;
  const bf16_t* b_base = B_TR ? job.B + (size_t)kbeg * p.ldb + n0 : job.B + (swf ? (size_t)0 : (size_t)n0 * p.ldb) + kbeg;
  const size_t a_step = A_TR ? (size_t)BK * p.lda : (size_t)BK;
  const size_t b_step = B_TR ? (size_t)BK * p.ldb : (size_t)BK;
  sa.load(a_base, p.lda, kend - kbeg, tid);
  sb.load(b_base, p.ldb, kend - kbeg, tid);
  sa.store(smem);
  sb.store(smem + 2 * A_TILE);
  if (kbeg + BK < kend) {
    // same issue order as in the steady-state loop (part by part, A then B): the compiler's
    // wait-count bookkeeping merges this order with the loop's at the loop header, and any
    // difference makes the loop wait for younger loads than the one it stores
    constexpr int PA0 = Stage<BM, NT, A_TR, KTAIL>::PER, PB0 = Stage<BN, NT, B_TR, KTAIL>::PER;
#pragma unroll
    for (int ks = 0; ks < BK / 32; ++ks) {
#pragma unroll
      for (int i = 0; i < PA0; ++i) sa.load_one(ks * PA0 + i, a_base + a_step, p.lda, kend - kbeg - BK, tid);
#pragma unroll
      for (int i = 0; i < PB0; ++i) sb.load_one(ks * PB0 + i, b_base + b_step, p.ldb, kend - kbeg - BK, tid);
    }
  }
  __syncthreads();

  // one slice; NEXT1: the registers hold a slice to park, NEXT2: one more to fetch.
  // The flags are compile-time so that the steady-state loop body is branch-free
  // (the wait-count bookkeeping of the loads then stays exact across iterations).
  // Fragments.  A k-step (k = 32) is FM x FN MFMAs, row block i outermost: all FN B fragments
  // of a step are live (two register sets: the next step's are requested while this one runs),
  // the A fragments pass through a ring of four (the one for row block g+2 is requested when
  // row block g starts).  The last row block of a slice is held back: its operands are in
  // registers, so its MFMAs run AFTER the barrier that ends the slice and cover the LDS latency
  // of the next slice's first fragments.
  constexpr int KS32 = BK / 32, ROWS = KS32 * FM;
  static_assert(ROWS % 4 == 0, "the A ring continues across slices");
  bf16x8 ar[4], bfr[2][FN];
  auto pending_row = [&](auto&& between) {
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      mfma16(acc[FM - 1][j], bfr[(KS32 - 1) & 1][j], ar[(ROWS - 1) % 4]);
      between(j);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto slice = [&](auto next1_t, auto next2_t, auto pend_t, int k0, int cur) {
    constexpr bool NEXT1 = decltype(next1_t)::value, NEXT2 = decltype(next2_t)::value;
    constexpr bool PEND = decltype(pend_t)::value;
    const bf16_t* a_lds = smem + cur * A_TILE;
    const bf16_t* b_lds = smem + 2 * A_TILE + cur * B_TILE;
    bf16_t* a_nxt = smem + (cur ^ 1) * A_TILE;
    bf16_t* b_nxt = smem + 2 * A_TILE + (cur ^ 1) * B_TILE;
    auto a_frag = [&](int g) {
      const int ks = g / FM, r0 = wm * TM + (g % FM) * 16;
      return A_TR ? tr_fragment16<BM>(a_lds, r0, ks * 32, lane) : kc_fragment16(a_lds, r0, ks, lane);
    };
    auto b_frag = [&](int ks, int j) {
      const int r0 = wn * TN_ + j * 16;
      return B_TR ? tr_fragment16<BN>(b_lds, r0, ks * 32, lane) : kc_fragment16(b_lds, r0, ks, lane);
    };
    // the first MFMA of the slice waits for two fragments only: keep this request order
    ar[0] = a_frag(0);
    bfr[0][0] = b_frag(0, 0);
    __builtin_amdgcn_sched_barrier(0);
    auto head_rest = [&](int n) {          // the other FN fragments of the head, one per call
      if (n + 1 < FN) bfr[0][n + 1] = b_frag(0, n + 1);
      else ar[1] = a_frag(1);
    };
    if (PEND) {
      pending_row(head_rest);
    } else {
#pragma unroll
      for (int n = 0; n < FN; ++n) head_rest(n);
      __builtin_amdgcn_sched_barrier(0);
    }
    // The other memory operations of a k-step -- the B fragment reads of the next step, the LDS
    // parks of this step's share of slice j+1 and the global loads that re-arm the same
    // registers with slice j+2 -- are dealt out evenly over the MFMAs and pinned there with
    // scheduling barriers so that they issue in the shadow of the matrix pipeline.
    constexpr int PA = Stage<BM, NT, A_TR, KTAIL>::PER, PB = Stage<BN, NT, B_TR, KTAIL>::PER;
    const bf16_t* a_g2 = a_base + (size_t)((k0 - kbeg) / BK + 2) * a_step;   // slice j+2
    const bf16_t* b_g2 = b_base + (size_t)((k0 - kbeg) / BK + 2) * b_step;
    const int k_left2 = kend - k0 - 2 * BK;
#pragma unroll
    for (int ks = 0; ks < KS32; ++ks) {
      const int nb = (ks + 1) & 1;
      const bool last = ks + 1 == KS32;
      // the last k-step has no fragments of a next step to fetch and one row block fewer to deal over
      const int SLOTS = last ? (FM - 1) * FN : FM * FN;
      const int FIRST = last ? FN : 0;                      // first op index of this step
      const int NOPS = FN + 2 * (PA + PB) - FIRST;
#pragma unroll
      for (int t = 0; t < SLOTS; ++t) {
        const int i = t / FN, j = t % FN, g = ks * FM + i;
        // operands swapped: the accumulator holds C^T blocks (see the epilogue)
        if (!PEND && ks == 0) mfma16_first(acc[i][j], bfr[ks & 1][j], ar[g % 4]);   // first slice of the tile
        else mfma16(acc[i][j], bfr[ks & 1][j], ar[g % 4]);
        if (j == 0 && g + 2 < ROWS) ar[(g + 2) % 4] = a_frag(g + 2);
#pragma unroll
        for (int oo = t * NOPS / SLOTS; oo < (t + 1) * NOPS / SLOTS; ++oo) {
          const int o = oo + FIRST;
          if (o < FN) {
            bfr[nb][o] = b_frag(ks + 1, o);
          } else if (o < FN + PA) {
            if (NEXT1) sa.store_one(ks * PA + (o - FN), a_nxt);
          } else if (o < FN + PA + PB) {
            if (NEXT1) sb.store_one(ks * PB + (o - FN - PA), b_nxt);
          } else if (o < FN + 2 * PA + PB) {
            if (NEXT2) sa.load_one(ks * PA + (o - FN - PA - PB), a_g2, p.lda, k_left2, tid);
          } else {
            if (NEXT2) sb.load_one(ks * PB + (o - FN - 2 * PA - PB), b_g2, p.ldb, k_left2, tid);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
  };
  using yes = std::true_type;
  using no = std::false_type;
  {
    // the first slice has no row block pending; the flags of the steady-state slices are
    // compile-time constants, so the loop body is branch-free
    int cur = 0, k0 = kbeg;
    if (k0 + 2 * BK < kend) {
      slice(yes{}, yes{}, no{}, k0, cur); k0 += BK; cur ^= 1;
      for (; k0 + 2 * BK < kend; k0 += BK, cur ^= 1) slice(yes{}, yes{}, yes{}, k0, cur);
      slice(yes{}, no{}, yes{}, k0, cur); k0 += BK; cur ^= 1;
      slice(no{}, no{}, yes{}, k0, cur);
    } else if (k0 + BK < kend) {
      slice(yes{}, no{}, no{}, k0, cur); k0 += BK; cur ^= 1;
      slice(no{}, no{}, yes{}, k0, cur);
    } else {
      slice(no{}, no{}, no{}, k0, cur);
    }
  }

  // epilogue; its staging strips overlay the slice buffers, free after the last barrier
  gemm_epilogue<EPI, FM, FN>(p, acc, reinterpret_cast<float*>(smem_raw) + wave * epilogue_stage_floats<FN>(), lane,
                             n0 + wn * TN_, job.tn * (BN / 2) + wn * (TN_ / 2), job.split, job.c_off,
                             m0 + BM <= p.M && n0 + BN <= p.N, [&](int i) { return m0 + wm * TM + i * 16; },
                             [&] { pending_row([](int) {}); });
}

template <bool A_TR, bool B_TR, int EPI, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_mfma_kernel(GemmParams p) {
  small_tile<A_TR, B_TR, EPI, KTAIL>(p, blockIdx.x);
}

// An input gradient (NN, whole slices) and a weight gradient (TN) that do not depend on one another in one grid: on few
// rows each alone leaves half of the chip's slots idle and costs a launch.  Blocks of a vision encoder, three such pairs
// each: 256 rows 207 -> 193 us, 577 rows 260 -> 241, 1500 rows 340 -> 323, 3000 rows 500 -> 485.
template <int EPI_NN, int EPI_TN, bool KTAIL>
__global__ __launch_bounds__(256) void gemm_joint_kernel(GemmParams nn, GemmParams tn, int nn_wgs) {
  if ((int)blockIdx.x < nn_wgs) small_tile<false, true, EPI_NN, false>(nn, blockIdx.x);
  else small_tile<true, true, EPI_TN, KTAIL>(tn, blockIdx.x - nn_wgs);
}

__device__ inline void splitk_reduce(const float* __restrict__ partial, int splits, int M, int N, float* __restrict__ C,
                                     int ldc, long i) {
  if (i >= (long)M * N) return;
  const int m = (int)(i / N), n = (int)(i % N);
  float4 s = {0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < splits; ++k) {
    float4 v = *reinterpret_cast<const float4*>(partial + (size_t)k * M * N + i);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  float* c = C + (size_t)m * ldc + n;
  c[0] += s.x; c[1] += s.y; c[2] += s.z; c[3] += s.w;
}
__global__ void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int M, int N,
                                     float* __restrict__ C, int ldc) {
  splitk_reduce(partial, splits, M, N, C, ldc, ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4);
}
// the split parts of a shared grid; blockIdx.y is the part
__global__ void splitk_reduce_parts_kernel(TnParts g) {
  const TnParts::Part& q = g.part[blockIdx.y];
  if (q.splits > 1) splitk_reduce(q.partial, q.splits, q.M, q.N, q.C, q.ldc, ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4);
}

// C = sum of the k ranges' partial products (+bias) (+residual), in range order
template <bool F32>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const float* __restrict__ partial, int splits, int M, int N,
                                                            void* __restrict__ C, int ldc, const bf16_t* __restrict__ bias,
                                                            const bf16_t* __restrict__ residual) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 8;
  if (i >= (long)M * N) return;
  const int m = (int)(i / N), n = (int)(i % N);
  float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < splits; ++k) {
    const float* q = partial + (size_t)k * M * N + i;
    const f32x4 lo = *reinterpret_cast<const f32x4*>(q), hi = *reinterpret_cast<const f32x4*>(q + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { v[e] += lo[e]; v[4 + e] += hi[e]; }
  }
  if (bias) {
    float b[8];
    load16(bias + n, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += b[e];
  }
  const size_t idx = (size_t)m * ldc + n;
  if (residual) {
    float r[8];
    load16(residual + idx, r);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += r[e];
  }
  if (F32) {
    *reinterpret_cast<f32x4*>((float*)C + idx) = f32x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<f32x4*>((float*)C + idx + 4) = f32x4{v[4], v[5], v[6], v[7]};
  } else {
    store16((bf16_t*)C + idx, v);
  }
}

// big_rows > 0: that many rows of 256x256 tiles, the other rows on 128x256 (tiles_m counts both)
struct Plan { int bm, bn, tiles_m, tiles_n, splits, k_per_split, big_rows = 0; };

constexpr int NUM_CU = 256;

// Tile and k split from a small cost model in microseconds.  A slice of k = 64 takes t_min when the chip is
// nearly empty and t_full when every slot works (the matrix pipe's power budget, shared by the active CUs), in
// between t_full * (share of busy slots)^power; a workgroup adds t_fixed.  A contraction that ends inside a slice adds
// t_cut; the 128x128 kernel tests every chunk of every slice for it instead (CUT_SMALL).  f_tn: a slice with both
// operands transposed against one with none.  A weight gradient reads and writes its fp32 C at 5.2 TB/s, a share
// `hidden` of which runs under the slices of others -- most where a CU holds two workgroups, so that short
// contractions want the smallest tile (TN 12288x3072 over 128 rows: 83 us with 256x256 tiles, 70 with 128x128; over
// 1536 rows 154 both).  A split writes and reads fp32 partial tiles at 8 TB/s (they stay in the memory-side
// cache) and costs one more launch (TN 8x1024 over 802 rows: 12.1 us, in three ranges 9.0).
// Measured on 527 shapes (blocks of 1024 to 4096 columns at 300 to 16384 rows, shapes drawn over the same range, and
// gradients of 8 to 128 conditions; every tile, splits 1-32): the plan it picks takes 1.2 % longer than the best one on
// average, 23 % at worst.
// The constants of weight gradients are those of a kernel that is gone: slices of 256x256 tiles are cut along k by now (a lone one takes
// 0.96 / 0.87 = 1.10 of an NT slice, f_tn says 1.13) and C goes through whole lines, which took 1-7 % off all fp32 epilogues.  So on shapes
// near a line the plan, the shared launch of two weight gradients and joint_plan still price a 256x256 tile a few per cent too
// high and may take a choice that is that much slower than the best; the table has not been refitted.
struct TileKind { int bm, bn, slots; double t_min, t_full, power, t_fixed, t_cut, f_tn, hidden; };
constexpr TileKind TILE_KINDS[] = {
  {256, 256, NUM_CU, 0.87, 1.36, 0.6, 5.5, 3.6, 1.13, 0.23},
  {128, 256, NUM_CU, 0.55, 0.77, 0.5, 4.0, 2.3, 1.34, 0.27},
  {256, 128, NUM_CU, 0.55, 0.77, 0.5, 4.0, 2.3, 1.34, 0.27},
  {128, 128, 2 * NUM_CU, 0.45, 0.92, 0.0, 3.4, 0.0, 1.12, 0.53},       // two workgroups per CU
};
constexpr double CUT_SMALL = 1.33;

// Splits of 2, 4 or 8 can be pinned to XCDs (see split_tile_of_block).
bool xcd_split_possible(int tiles, int splits) {
  return (splits == 2 || splits == 4 || splits == 8) && tiles % (8 / splits) == 0;
}

// one grid of `wgs` workgroups that each walk `per` slices
double grid_time(const TileKind& tk, int layout, bool cut, long wgs, int per) {
  const bool small = tk.bm == 128 && tk.bn == 128;
  const double f = (layout == GEMM_NT ? 1.0 : layout == GEMM_NN ? 1.05 : tk.f_tn) * (small && cut ? CUT_SMALL : 1.0);
  const double fixed = tk.t_fixed + (cut ? tk.t_cut : 0.0);
  const long full = wgs / tk.slots, rest = wgs % tk.slots;
  double t = full * (per * tk.t_full * f + fixed);
  if (rest) {
    const double u = (double)rest / tk.slots;
    double ts;
    if (small) ts = u <= 0.5 ? tk.t_min : tk.t_min + (tk.t_full - tk.t_min) * std::sqrt(2.0 * u - 1.0);
    else ts = std::max(tk.t_min, tk.t_full * std::pow(u, tk.power));
    t += per * ts * f + fixed;
  }
  return t;
}
// ... and its output of mn elements: the partial tiles of a split and their reduction, or a weight gradient's C
double output_time(const TileKind& tk, int layout, int splits, double mn, double grid) {
  if (splits > 1) return layout == GEMM_TN ? 2.4 + (splits + 1) * mn / 1e6 : 4.5 + (4 * splits + 1) * mn / 4e6;
  if (layout != GEMM_TN) return 0.0;
  const double c = mn * 8.0 / 5.2e6;
  return c - tk.hidden * std::min(c, grid);
}

// Most k ranges a plan may use.  Weight gradient: as many as fill the chip with 256x256 tiles, four
// slices each at least -- a bound that only grows with K, so that a workspace sized for the longest
// pack serves every shorter one.  The other layouts split only products of few rows.
int split_cap(int layout, int M, int N, int K) {
  const int slices = cdiv(K, BK);
  long cap = slices / 4;
  if (layout == GEMM_TN) cap = std::min<long>(cap, NUM_CU / ((long)cdiv(M, 256) * cdiv(N, 256)));
  else cap = std::min<long>(cap, std::min(SPLIT_ROWS_MAX / M, 16));
  return cap < 1 ? 1 : (int)std::min<long>(cap, 32);
}

// Rows on tiles of two heights: as many 256-row tiles as fill whole rounds (or all that the rows fill), the other rows on
// 128-row tiles, which run beside the last of the former and behind them.  us against the best of the four tiles: NT 5477x3072x1024
// 46 -> 40, 5477x4096x1024 51 -> 46, 777x22016x4096 161 -> 143, 8192x4608x1152 83 -> 76, 6352x6144x4096 244 -> 230, NN 1783x12288x3072 128 -> 110,
// 8192x11008x4096 527 -> 516.  Of 260 products of 384 to 16384 rows that it takes (operands out of the caches) five
// are 2 to 3 % slower (NT 4509x12216x6160, 8527x9608x4456: ragged columns and a long contraction), the mean is 8 % faster.
// Where 128x128 is the best of the four it competes only from six slices on and with columns that fill whole cache lines: below, a
// second workgroup on the CU hides the output, which the model prices lower than it is.  71 products of ragged columns took 6 %
// longer with two heights on average and up to 23 % (NT 2566x13424x200 34 -> 40, NN 11265x4816x176 45 -> 55); of 127 of four and five
// slices 34 took 2 to 13 % longer (NT 8205x4096x224 31.4 -> 35.6), of 16 shorter ones twelve (NN 1469x12288x128 12.7 -> 14.2).  Of 135
// from six slices on seven took 2 to 7 % longer, the mean is 4 % faster (NT 2238x9216x400 29 -> 25).
void mixed_rows(int layout, int M, int N, int K, Plan* best, double* best_t) {
  const TileKind &big = TILE_KINDS[0], &low = TILE_KINDS[1];
  const int tiles_n = cdiv(N, 256), slices = cdiv(K, BK);
  if (N < 256 || M < 256 + 128) return;
  if (best->bm == 128 && best->bn == 128 && (slices < 6 || N % 64)) return;
  const bool cut = K % BK;
  const double f = layout == GEMM_NT ? 1.0 : 1.05, fixed_cut = cut ? 1.0 : 0.0;
  const double t_big = slices * big.t_full * f + big.t_fixed + fixed_cut * big.t_cut;
  const double t_low = slices * low.t_full * f + low.t_fixed + fixed_cut * low.t_cut;
  auto consider = [&](long rows) {
    const long low_rows = cdiv(M - rows * 256, 128L);
    if (rows < 1 || rows * 256 >= M || low_rows < 1) return;
    const long wgs = rows * tiles_n, rest = wgs % NUM_CU;
    long lows = low_rows * tiles_n;
    double t = wgs / NUM_CU * t_big;
    if (rest) {
      // the last round of the big ones, with low ones on the CUs they leave
      const long beside = std::min(lows, (NUM_CU - rest) * std::max(1L, (long)(t_big / t_low)));
      t += beside > 0 && rest + beside >= NUM_CU * 3 / 4 ? t_big : grid_time(big, layout, cut, std::min<long>(NUM_CU, rest + beside), slices);
      lows -= beside;
    }
    if (lows > 0) t += grid_time(low, layout, cut, lows, slices);
    if (t < *best_t) {
      *best_t = t;
      *best = Plan{256, 256, (int)(rows + low_rows), tiles_n, 1, slices * BK, (int)rows};
    }
  };
  const long full = M / 256, rounds = full * tiles_n / NUM_CU;
  consider(full);
  if (rounds >= 1) consider(rounds * NUM_CU / tiles_n);
  if (rounds >= 2) consider((rounds - 1) * NUM_CU / tiles_n);
  else if (tiles_n < NUM_CU) consider(full / 2);
}

Plan make_plan(int layout, int M, int N, int K, size_t partial_bytes, bool may_split, double* time = nullptr) {
  Plan best{};
  double best_t = 1e30;
  const int slices = cdiv(K, BK), cap = may_split ? split_cap(layout, M, N, K) : 1;
  const double mn = (double)M * N;
  for (const TileKind& tk : TILE_KINDS) {
    const long tiles = (long)cdiv(M, tk.bm) * cdiv(N, tk.bn);
    for (int sp = 1; sp <= cap; ++sp) {
      const int per = cdiv(slices, sp);
      if (cdiv(slices, per) != sp) continue;
      if (sp > 1 && sp * mn * sizeof(float) > (double)partial_bytes) break;
      double t = grid_time(tk, layout, K % BK != 0, tiles * sp, per);
      t += output_time(tk, layout, sp, mn, t);
      if (xcd_split_possible((int)tiles, sp)) t *= 0.97;
      if (t < best_t) {
        best_t = t;
        best.bm = tk.bm; best.bn = tk.bn;
        best.tiles_m = cdiv(M, tk.bm); best.tiles_n = cdiv(N, tk.bn);
        best.splits = sp; best.k_per_split = per * BK;
      }
    }
  }
  if (layout != GEMM_TN) mixed_rows(layout, M, N, K, &best, &best_t);
  if (time) *time = best_t;
  return best;
}

template <bool A_TR, bool B_TR, int EPI, bool KTAIL>
bm_status launch_k(const GemmParams& p, hipStream_t st) {
  constexpr size_t lds = (size_t)2 * (128 + 128) * BK * sizeof(bf16_t);
  static_assert(lds >= 4 * epilogue_stage_floats<4>() * sizeof(float), "the epilogue's strips overlay the slices");
  auto kern = gemm_mfma_kernel<A_TR, B_TR, EPI, KTAIL>;
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_relaxed)) {
    BM_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_done.store(true, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n * p.splits * p.grid_groups), dim3(256), lds, st, p);
  BM_CHECK_LAUNCH("gemm_mfma");
  return BM_OK;
}

// the zero-filling variant only when a k range is not a whole number of slices
template <bool A_TR, bool B_TR, int EPI>
bm_status launch(const GemmParams& p, hipStream_t st) {
  if (p.K % BK) return launch_k<A_TR, B_TR, EPI, true>(p, st);
  return launch_k<A_TR, B_TR, EPI, false>(p, st);
}

// 128x128 tiles
bm_status launch_small(int layout, const GemmParams& p, hipStream_t st) {
  if (layout == GEMM_TN)
    return p.splits > 1 ? launch<true, true, EPI_PARTIAL>(p, st) : launch<true, true, EPI_ADD>(p, st);
  if (layout == GEMM_NT) {
    if (p.splits > 1) return launch<false, false, EPI_PARTIAL>(p, st);
    if (p.swf_a) return launch<false, false, EPI_SWIGLU_FWD>(p, st);
    return p.residual ? launch<false, false, EPI_RES>(p, st) : launch<false, false, EPI_PLAIN>(p, st);
  }
  if (p.splits > 1) return launch<false, true, EPI_PARTIAL>(p, st);
  if (p.sw_up) return launch<false, true, EPI_SWIGLU_BWD>(p, st);
  return p.residual ? launch<false, true, EPI_RES>(p, st) : launch<false, true, EPI_PLAIN>(p, st);
}

}  // namespace

bool gemm_mfma_supported(int layout, int dtype, int M, int N, int K, int lda, int ldb, int ldc,
                         const GemmEpilogue& epi) {
  (void)epi;
  if (dtype != BM_DTYPE_BF16) return false;
  if (lda % 8 || ldb % 8) return false;                  // 16-byte rows
  if (N < 64) return false;                              // tiny problems: generic kernel
  if (layout == GEMM_TN) {
    // operands are [k][row]: rows come in chunks of 8, any k range of at least one chunk
    // works (a short one is zero-filled); one of M and K may be small (the 8..32-row
    // products of the adaLN modulation), not both
    if (M % 8 || N % 8 || ldc % 4) return false;
    return M >= 8 && K >= 8 && (M >= 64 || K >= 64);
  }
  // row-major A: rows past M are clamped to the last one and never stored, so few rows are fine
  if (M < 1 || K < 64) return false;
  return K % 8 == 0 && N % 8 == 0 && ldc % 8 == 0;          // 16-byte row chunks of C
}

size_t gemm_mfma_scratch_bytes(int layout, int M, int N, int K) {
  if (layout == GEMM_TN) {
    const int cap = split_cap(layout, M, N, K);
    return cap > 1 ? (size_t)cap * M * N * sizeof(float) : 0;
  }
  const Plan pl = make_plan(layout, M, N, K, ~(size_t)0, true);
  return pl.splits > 1 ? (size_t)pl.splits * M * N * sizeof(float) : 0;
}

void gemm_mfma_plan(int layout, int M, int N, int K, size_t scratch_bytes, int* bm, int* bn, int* splits) {
  const Plan pl = make_plan(layout, M, N, K, scratch_bytes, true);
  *bm = pl.big_rows > 0 ? 256 + 128 : pl.bm; *bn = pl.bn; *splits = pl.splits;
}

bm_status gemm_mfma(int layout, int M, int N, int K, const void* A, int lda, const void* B, int ldb,
                    void* C, int ldc, const GemmEpilogue& epi, void* scratch, size_t scratch_bytes,
                    hipStream_t st) {
  // the k range is split as far as the workspace allows; a fused activation needs the whole sum at once.  NT and NN
  // need no workspace, so one that is not aligned for the partial tiles counts as none.
  if (layout != GEMM_TN && reinterpret_cast<uintptr_t>(scratch) % 16) scratch_bytes = 0;
  const Plan pl = make_plan(layout, M, N, K, scratch ? scratch_bytes : 0, !epi.swiglu_up && !epi.swiglu_fwd_a);
  GemmParams p;
  p.A = (const bf16_t*)A; p.B = (const bf16_t*)B; p.C = C;
  p.bias = (const bf16_t*)epi.bias; p.residual = (const bf16_t*)epi.residual;
  p.partial = (float*)scratch;
  p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldc = ldc;
  p.tiles_m = pl.tiles_m; p.tiles_n = pl.tiles_n; p.splits = pl.splits; p.k_per_split = pl.k_per_split;
  p.out_fp32 = epi.out_fp32;
  p.sw_up = (const bf16_t*)epi.swiglu_up; p.sw_dup = (bf16_t*)epi.swiglu_dup; p.sw_a = (bf16_t*)epi.swiglu_a;
  p.swf_a = (bf16_t*)epi.swiglu_fwd_a;
  if (p.swf_a && (layout != GEMM_NT || N % 256 || epi.bias || epi.residual || epi.out_fp32)) {
    set_error("gemm: the SwiGLU forward epilogue needs the NT layout, N a multiple of 256 and no bias");
    return BM_ERR_INVALID_ARG;
  }
  p.tile_group = nullptr; p.group_rows = nullptr; p.row_tiles = nullptr; p.source = nullptr; p.src_rows = 0; p.row_scale = nullptr; p.row_dot = nullptr; p.b_group_stride = 0; p.c_group_stride = 0;
  p.grid_groups = 1;
  p.xcd_split = xcd_split_possible(pl.tiles_m * pl.tiles_n, pl.splits) ? 1 : 0;
  p.big_rows = pl.big_rows;
  BM_RETURN_IF(pl.big_rows > 0 ? launch_gemm_alt_mixed(layout, p, st)
               : pl.bm == 128 && pl.bn == 128 ? launch_small(layout, p, st) : launch_gemm_alt(layout, pl.bm, pl.bn, p, st));
  if (pl.splits > 1 && layout == GEMM_TN) {
    hipLaunchKernelGGL(splitk_reduce_kernel, dim3(cdiv((long)M * N / 4, 256)), dim3(256), 0, st,
                       (const float*)scratch, pl.splits, M, N, (float*)C, ldc);
    BM_CHECK_LAUNCH("splitk_reduce");
  } else if (pl.splits > 1) {
    auto kern = epi.out_fp32 ? splitk_finish_kernel<true> : splitk_finish_kernel<false>;
    hipLaunchKernelGGL(kern, dim3(cdiv((long)M * N / 8, 256)), dim3(256), 0, st, (const float*)scratch, pl.splits, M, N,
                       C, ldc, (const bf16_t*)epi.bias, (const bf16_t*)epi.residual);
    BM_CHECK_LAUNCH("splitk_finish");
  }
  return BM_OK;
}

// Most k ranges of a paired launch (0: the pair does not qualify).  As split_cap(), it only grows with K.
static int pair_split_cap(int K, int M0, int N0, int M1, int N1) {
  if (M0 < 256 || N0 < 256 || M1 < 256 || N1 < 256) return 0;
  const long tiles = (long)cdiv(M0, 256) * cdiv(N0, 256) + (long)cdiv(M1, 256) * cdiv(N1, 256);
  return (int)std::min<long>(std::min<long>(NUM_CU / tiles, 32), cdiv(K, BK) / 4);
}

// the number of ranges it takes: the most that a whole number of slices each comes to
static int pair_splits(int K, int M0, int N0, int M1, int N1) {
  const int slices = cdiv(K, BK);
  int sp = pair_split_cap(K, M0, N0, M1, N1);
  for (; sp >= 1; --sp)
    if (cdiv(slices, cdiv(slices, sp)) == sp) break;
  return sp;
}

size_t gemm_mfma_tn_pair_scratch_bytes(int K, int M0, int N0, int M1, int N1) {
  const int sp = pair_split_cap(K, M0, N0, M1, N1);
  if (sp <= 1) return 0;
  return align_up((size_t)sp * M0 * N0 * sizeof(float), 256) + (size_t)sp * M1 * N1 * sizeof(float);
}

namespace {

TnParts::Part tn_part(const GemmCall& w, const Plan& pl, float* partial, int first_wg) {
  TnParts::Part q;
  q.A = (const bf16_t*)w.A; q.B = (const bf16_t*)w.B; q.C = (float*)w.C; q.partial = partial;
  q.M = w.M; q.N = w.N; q.K = w.K; q.lda = w.lda; q.ldb = w.ldb; q.ldc = w.ldc;
  q.tiles_m = pl.tiles_m; q.tiles_n = pl.tiles_n; q.splits = pl.splits; q.k_per_split = pl.k_per_split;
  // (split tiles are pinned to XCDs by the id of a workgroup in its grid)
  q.xcd_split = first_wg % 8 == 0 && xcd_split_possible(pl.tiles_m * pl.tiles_n, pl.splits) ? 1 : 0;
  q.first_wg = first_wg;
  return q;
}

bm_status launch_tn_parts(const TnParts& g, hipStream_t st) {
  BM_RETURN_IF(launch_gemm_alt_tn_parts(g, st));
  long longest = 0, last = g.n - 1;                            // unsplit parts come first
  for (int i = 0; i < g.n; ++i)
    if (g.part[i].splits > 1) { longest = std::max(longest, (long)g.part[i].M * g.part[i].N); last = std::min<long>(last, i); }
  if (longest == 0) return BM_OK;
  TnParts split = g;
  split.n = g.n - (int)last;
  for (int i = 0; i < split.n; ++i) split.part[i] = g.part[last + i];
  hipLaunchKernelGGL(splitk_reduce_parts_kernel, dim3(cdiv(longest / 4, 256), split.n), dim3(256), 0, st, split);
  BM_CHECK_LAUNCH("splitk_reduce");
  return BM_OK;
}

}  // namespace

// Two weight gradients C_i[M_i,N_i] += A_i[K,M_i]^T B_i[K,N_i] over the same K in ONE grid, when
// both plans use 256x256 tiles and whole slices: a gradient whose tiles x splits do not fill
// the chip (1024x1024 next to 3072x1024 in a ViT-L block) no longer has the machine to itself.
// Returns false (nothing launched) when the pair does not qualify; the caller then runs two GEMMs.
bool gemm_mfma_tn_pair(int K, int M0, int N0, const void* A0, int lda0, const void* B0, int ldb0, void* C0, int ldc0,
                       int M1, int N1, const void* A1, int lda1, const void* B1, int ldb1, void* C1, int ldc1,
                       void* scratch, size_t scratch_bytes, hipStream_t st, bm_status* rc, double* time) {
  // rc == nullptr: only answer whether the pair qualifies
  const GemmEpilogue none;
  if (rc) *rc = BM_OK;
  if (!gemm_mfma_supported(GEMM_TN, BM_DTYPE_BF16, M0, N0, K, lda0, ldb0, ldc0, none) ||
      !gemm_mfma_supported(GEMM_TN, BM_DTYPE_BF16, M1, N1, K, lda1, ldb1, ldc1, none)) return false;
  // one plan for both: 256x256 tiles and the largest common k split whose workgroups fit the chip
  // in one round, so that all of them run equally long; it must beat the two separate plans
  const int sp = pair_splits(K, M0, N0, M1, N1);
  if (sp < 1) return false;
  const int slices = cdiv(K, BK);
  Plan a{}, b{};
  a.bm = a.bn = b.bm = b.bn = 256;
  a.tiles_m = cdiv(M0, 256); a.tiles_n = cdiv(N0, 256);
  b.tiles_m = cdiv(M1, 256); b.tiles_n = cdiv(N1, 256);
  a.splits = b.splits = sp;
  a.k_per_split = b.k_per_split = cdiv(slices, sp) * BK;
  {
    double t0, t1;
    make_plan(GEMM_TN, M0, N0, K, scratch_bytes, true, &t0);
    make_plan(GEMM_TN, M1, N1, K, scratch_bytes, true, &t1);
    const double mn0 = (double)M0 * N0, mn1 = (double)M1 * N1;
    double together = grid_time(TILE_KINDS[0], GEMM_TN, K % BK != 0,
                                ((long)a.tiles_m * a.tiles_n + (long)b.tiles_m * b.tiles_n) * sp, cdiv(slices, sp));
    if (sp > 1) together += output_time(TILE_KINDS[0], GEMM_TN, sp, mn0, 0.0) + output_time(TILE_KINDS[0], GEMM_TN, sp, mn1, 0.0);
    else together += output_time(TILE_KINDS[0], GEMM_TN, 1, mn0 + mn1, together);
    if (together >= t0 + t1) return false;
    if (time) *time = together;
  }
  const size_t part0 = a.splits > 1 ? align_up((size_t)a.splits * M0 * N0 * sizeof(float), 256) : 0;
  const size_t part1 = b.splits > 1 ? (size_t)b.splits * M1 * N1 * sizeof(float) : 0;
  if (part0 + part1 > scratch_bytes || (part0 + part1 > 0 && !scratch)) return false;
  const int wgs0 = a.tiles_m * a.tiles_n * a.splits;
  const bool xa = xcd_split_possible(a.tiles_m * a.tiles_n, a.splits), xb = xcd_split_possible(b.tiles_m * b.tiles_n, b.splits);
  if (xb && wgs0 % 8) return false;               // the second problem's XCD pinning needs an aligned start
  if (!rc) return true;
  TnParts g;
  g.n = 2;
  g.one_list = 0;
  g.part[0] = tn_part(GemmCall{M0, N0, K, A0, lda0, B0, ldb0, C0, ldc0}, a, (float*)scratch, 0);
  g.part[1] = tn_part(GemmCall{M1, N1, K, A1, lda1, B1, ldb1, C1, ldc1}, b, (float*)((char*)scratch + part0), wgs0);
  *rc = launch_tn_parts(g, st);
  return true;
}

// ---- all weight gradients of a block in one grid
//
// They are ready one after the other, and alone each leaves CUs idle or splits its k range: a block of 1024 columns is
// 48 + 16 + 64 + 64 tiles of 256x256.  Together those are one round of 192 without partial tiles; where a round has room
// for more, all are split alike, and the one gradient that would otherwise open a round of its own is split over its
// CUs.  A slice of 192 tiles takes 1.19 us, of 256 tiles 1.37 (power), so the idle quarter costs little.  Forward and backward of a block:
// vision encoder of 1024 columns, 3000 rows 508 -> 457 us, 5477 rows 816 -> 745, 16384 rows 1688 -> 1650; generator of 1152 columns,
// 8192 rows 1364 -> 1274; 256 columns, 8000 rows 242 -> 213; decoder of 2048 columns, 6000 rows 2180 -> 2111.
namespace {

struct TnGroupPlan { int split_part, splits, per; };          // the part that is split: NO_PART, ALL_PARTS or its index
constexpr int NO_PART = -1, ALL_PARTS = -2;

// `longer` workgroups of per0 slices each, then `shorter` ones of per1
double two_lengths_time(const TileKind& tk, bool cut, long longer, int per0, long shorter, int per1) {
  if (shorter == 0) return grid_time(tk, GEMM_TN, cut, longer, per0);
  const double fixed = tk.t_fixed + (cut ? tk.t_cut : 0.0);
  const double t0 = per0 * tk.t_full * tk.f_tn + fixed, t1 = per1 * tk.t_full * tk.f_tn + fixed;
  const long rest = longer % tk.slots;
  if (rest) shorter = std::max(0L, shorter - (tk.slots - rest) * (long)(t0 / t1));       // beside the last of the long ones
  return cdiv(longer, (long)tk.slots) * t0 + (shorter ? grid_time(tk, GEMM_TN, cut, shorter, per1) : 0.0);
}

bool tn_group_plan(const GemmCall* w, int n, size_t scratch_bytes, TnGroupPlan* plan, double* time) {
  const TileKind& tk = TILE_KINDS[0];
  const GemmEpilogue none;
  if (n < 2 || n > TnParts::MAX) return false;
  const int K = w[0].K, slices = cdiv(K, BK);
  const bool cut = K % BK;
  long tiles[TnParts::MAX], all = 0;
  double mn = 0.0;
  for (int i = 0; i < n; ++i) {
    if (w[i].K != K || !gemm_mfma_supported(GEMM_TN, BM_DTYPE_BF16, w[i].M, w[i].N, K, w[i].lda, w[i].ldb, w[i].ldc, none)) return false;
    tiles[i] = (long)cdiv(w[i].M, 256) * cdiv(w[i].N, 256);
    all += tiles[i];
    mn += (double)w[i].M * w[i].N;
  }
  double best = grid_time(tk, GEMM_TN, cut, all, slices);
  best += output_time(tk, GEMM_TN, 1, mn, best);
  *plan = TnGroupPlan{NO_PART, 1, slices};
  for (int sp = 2; sp <= std::min<long>(std::min<long>(slices / 4, 32), NUM_CU / all); ++sp) {
    const int per = cdiv(slices, sp);
    if (cdiv(slices, per) != sp) continue;
    if (sp * mn * sizeof(float) + 256.0 * n > (double)scratch_bytes) break;
    const double t = grid_time(tk, GEMM_TN, cut, all * sp, per) + output_time(tk, GEMM_TN, sp, mn, 0.0);
    if (t < best) { best = t; *plan = TnGroupPlan{ALL_PARTS, sp, per}; }
  }
  for (int i = 0; i < n; ++i) {
    const double mni = (double)w[i].M * w[i].N;
    for (int sp = 2; sp <= split_cap(GEMM_TN, w[i].M, w[i].N, K); ++sp) {
      const int per = cdiv(slices, sp);
      if (cdiv(slices, per) != sp) continue;
      if (sp * mni * sizeof(float) > (double)scratch_bytes) break;
      double t = two_lengths_time(tk, cut, all - tiles[i], slices, tiles[i] * sp, per);
      t += output_time(tk, GEMM_TN, 1, mn - mni, t) + output_time(tk, GEMM_TN, sp, mni, t);
      if (t < best) { best = t; *plan = TnGroupPlan{i, sp, per}; }
    }
  }
  if (time) *time = best;
  return true;
}

}  // namespace

double gemm_mfma_tn_group_time(const GemmCall* w, int n, size_t scratch_bytes) {
  TnGroupPlan plan;
  double t;
  return tn_group_plan(w, n, scratch_bytes, &plan, &t) ? t : -1.0;
}

void gemm_mfma_tn_group_ranges(const GemmCall* w, int n, size_t scratch_bytes, int32_t* k_ranges) {
  TnGroupPlan plan;
  const bool shared = tn_group_plan(w, n, scratch_bytes, &plan, nullptr);
  for (int i = 0; i < n; ++i) k_ranges[i] = !shared ? 0 : plan.split_part == ALL_PARTS || plan.split_part == i ? plan.splits : 1;
}

int gemm_mfma_tn_pair_ranges(int K, int M0, int N0, int M1, int N1) { return pair_splits(K, M0, N0, M1, N1); }

bm_status gemm_mfma_tn_group(const GemmCall* w, int n, void* scratch, size_t scratch_bytes, hipStream_t st) {
  TnGroupPlan plan;
  if (!tn_group_plan(w, n, scratch ? scratch_bytes : 0, &plan, nullptr)) {
    set_error("gemm: these weight gradients share no launch");
    return BM_ERR_UNSUPPORTED;
  }
  TnParts g;
  g.n = 0;
  int first = 0;
  size_t part = 0;
  auto add = [&](int i, int splits, int per) {
    const Plan pl{256, 256, cdiv(w[i].M, 256), cdiv(w[i].N, 256), splits, per * BK, 0};
    g.part[g.n++] = tn_part(w[i], pl, (float*)((char*)scratch + part), first);
    first += pl.tiles_m * pl.tiles_n * splits;
    if (splits > 1) part += align_up((size_t)splits * w[i].M * w[i].N * sizeof(float), 256);
  };
  for (int i = 0; i < n; ++i)
    if (i != plan.split_part && plan.split_part != ALL_PARTS) add(i, 1, cdiv(w[i].K, BK));
  g.one_list = first <= NUM_CU ? first : 0;
  for (int i = 0; i < n; ++i)                                 // the shorter workgroups last
    if (i == plan.split_part || plan.split_part == ALL_PARTS) add(i, plan.splits, plan.per);
  return launch_tn_parts(g, st);
}

double gemm_mfma_time(int layout, const GemmCall& w, size_t scratch_bytes) {
  double t;
  make_plan(layout, w.M, w.N, w.K, scratch_bytes, true, &t);
  return t;
}

namespace {

// The k ranges of an input gradient (0) and a weight gradient (1) in one grid of 128x128 tiles that fits the chip's slots
// in one round, by the same model: the longest chain of slices at the rate of a nearly empty chip, or all slices at the
// rate of a full one.  false: separate launches are expected to be as fast (or the pair has more tiles than slots: from
// there on larger tiles are the better ones).
bool joint_plan(const GemmCall& nn, const GemmCall& tn, size_t scratch_bytes, Plan* pn, Plan* pt, double* time = nullptr) {
  const TileKind& tk = TILE_KINDS[3];
  const GemmEpilogue none;
  if (!gemm_mfma_supported(GEMM_NN, BM_DTYPE_BF16, nn.M, nn.N, nn.K, nn.lda, nn.ldb, nn.ldc, none) ||
      !gemm_mfma_supported(GEMM_TN, BM_DTYPE_BF16, tn.M, tn.N, tn.K, tn.lda, tn.ldb, tn.ldc, none) || nn.K % BK) return false;
  const long tiles0 = (long)cdiv(nn.M, 128) * cdiv(nn.N, 128), tiles1 = (long)cdiv(tn.M, 128) * cdiv(tn.N, 128);
  if (tiles0 + tiles1 > tk.slots) return false;
  double apart0, apart1;
  make_plan(GEMM_NN, nn.M, nn.N, nn.K, scratch_bytes, true, &apart0);
  make_plan(GEMM_TN, tn.M, tn.N, tn.K, scratch_bytes, true, &apart1);
  const int sl0 = cdiv(nn.K, BK), sl1 = cdiv(tn.K, BK);
  const int cap0 = split_cap(GEMM_NN, nn.M, nn.N, nn.K), cap1 = split_cap(GEMM_TN, tn.M, tn.N, tn.K);
  const double mn0 = (double)nn.M * nn.N, mn1 = (double)tn.M * tn.N;
  const double f0 = 1.05, f1 = tk.f_tn * (tn.K % BK ? CUT_SMALL : 1.0);
  double best = apart0 + apart1;
  bool found = false;
  for (int s0 = 1; s0 <= cap0 && tiles0 * s0 + tiles1 <= tk.slots; ++s0) {
    const int per0 = cdiv(sl0, s0);
    if (cdiv(sl0, per0) != s0) continue;
    const double part0 = s0 > 1 ? (double)align_up((size_t)(s0 * mn0 * sizeof(float)), 256) : 0.0;
    if (part0 > (double)scratch_bytes) break;
    for (int s1 = 1; s1 <= cap1 && tiles0 * s0 + tiles1 * s1 <= tk.slots; ++s1) {
      const int per1 = cdiv(sl1, s1);
      if (cdiv(sl1, per1) != s1) continue;
      if (s1 > 1 && part0 + s1 * mn1 * sizeof(float) > (double)scratch_bytes) break;
      const double chain = std::max(per0 * f0, per1 * f1) * tk.t_min;
      const double all = (tiles0 * s0 * per0 * f0 + tiles1 * s1 * per1 * f1) / tk.slots * tk.t_full;
      double t = std::max(chain, all) + tk.t_fixed;
      t += output_time(tk, GEMM_NN, s0, mn0, t) + output_time(tk, GEMM_TN, s1, mn1, t);
      if (t < best) {
        best = t; found = true;
        *pn = Plan{128, 128, cdiv(nn.M, 128), cdiv(nn.N, 128), s0, per0 * BK};
        *pt = Plan{128, 128, cdiv(tn.M, 128), cdiv(tn.N, 128), s1, per1 * BK};
      }
    }
  }
  if (time) *time = best;
  return found;
}

// all partial tiles of such a grid
constexpr size_t JOINT_PARTIAL_BYTES = (size_t)TILE_KINDS[3].slots * 128 * 128 * sizeof(float) + 256;

GemmParams plain_params(const GemmCall& g, const Plan& pl, float* partial) {
  GemmParams p;
  p.A = (const bf16_t*)g.A; p.B = (const bf16_t*)g.B; p.C = g.C; p.bias = nullptr; p.residual = nullptr;
  p.partial = partial;
  p.M = g.M; p.N = g.N; p.K = g.K; p.lda = g.lda; p.ldb = g.ldb; p.ldc = g.ldc;
  p.tiles_m = pl.tiles_m; p.tiles_n = pl.tiles_n; p.splits = pl.splits; p.k_per_split = pl.k_per_split;
  p.out_fp32 = 0;
  p.xcd_split = xcd_split_possible(pl.tiles_m * pl.tiles_n, pl.splits) ? 1 : 0;
  p.tile_group = nullptr; p.group_rows = nullptr; p.row_tiles = nullptr; p.source = nullptr; p.src_rows = 0; p.row_scale = nullptr; p.row_dot = nullptr; p.b_group_stride = 0; p.c_group_stride = 0; p.grid_groups = 1;
  return p;
}

template <int EPI_NN, int EPI_TN, bool KTAIL>
bm_status launch_joint(const GemmParams& nn, const GemmParams& tn, hipStream_t st) {
  constexpr size_t lds = (size_t)2 * (128 + 128) * BK * sizeof(bf16_t);
  auto kern = gemm_joint_kernel<EPI_NN, EPI_TN, KTAIL>;
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_relaxed)) {
    BM_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_done.store(true, std::memory_order_relaxed);
  }
  const int wgs0 = nn.tiles_m * nn.tiles_n * nn.splits, wgs1 = tn.tiles_m * tn.tiles_n * tn.splits;
  hipLaunchKernelGGL(kern, dim3(wgs0 + wgs1), dim3(256), lds, st, nn, tn, wgs0);
  BM_CHECK_LAUNCH("gemm_joint");
  return BM_OK;
}

}  // namespace

size_t gemm_nn_tn_scratch_bytes(size_t nn, size_t tn, int dtype) {
  return dtype == BM_DTYPE_BF16 ? std::min(nn + tn, JOINT_PARTIAL_BYTES) : 0;
}

double gemm_mfma_nn_tn_time(const GemmCall& nn, const GemmCall& tn, size_t scratch_bytes) {
  Plan pn, pt;
  double t;
  return joint_plan(nn, tn, scratch_bytes, &pn, &pt, &t) ? t : -1.0;
}

bool gemm_mfma_nn_tn_ranges(const GemmCall& nn, const GemmCall& tn, size_t scratch_bytes, int* nn_ranges, int* tn_ranges) {
  Plan pn, pt;
  if (!joint_plan(nn, tn, scratch_bytes, &pn, &pt)) return false;
  *nn_ranges = pn.splits; *tn_ranges = pt.splits;
  return true;
}

bool gemm_mfma_nn_tn(const GemmCall& nn, const GemmCall& tn, void* scratch, size_t scratch_bytes, hipStream_t st,
                     bm_status* rc) {
  if (!scratch || reinterpret_cast<uintptr_t>(scratch) % 16) scratch_bytes = 0;
  Plan pn, pt;
  if (!joint_plan(nn, tn, scratch_bytes, &pn, &pt)) return false;
  const size_t part0 = pn.splits > 1 ? align_up((size_t)pn.splits * nn.M * nn.N * sizeof(float), 256) : 0;
  float* partial1 = (float*)((char*)scratch + part0);
  const GemmParams a = plain_params(nn, pn, (float*)scratch), b = plain_params(tn, pt, partial1);
  auto launch_all = [&]() -> bm_status {
    ProfScope prof(PROF_GEMM_NN, 2.0 * nn.M * nn.N * nn.K + 2.0 * tn.M * tn.N * tn.K, st);     // the class of the first
    const bool cut = tn.K % BK;
    if (pn.splits > 1) {
      if (pt.splits > 1) BM_RETURN_IF((cut ? launch_joint<EPI_PARTIAL, EPI_PARTIAL, true>(a, b, st) : launch_joint<EPI_PARTIAL, EPI_PARTIAL, false>(a, b, st)));
      else BM_RETURN_IF((cut ? launch_joint<EPI_PARTIAL, EPI_ADD, true>(a, b, st) : launch_joint<EPI_PARTIAL, EPI_ADD, false>(a, b, st)));
    } else {
      if (pt.splits > 1) BM_RETURN_IF((cut ? launch_joint<EPI_PLAIN, EPI_PARTIAL, true>(a, b, st) : launch_joint<EPI_PLAIN, EPI_PARTIAL, false>(a, b, st)));
      else BM_RETURN_IF((cut ? launch_joint<EPI_PLAIN, EPI_ADD, true>(a, b, st) : launch_joint<EPI_PLAIN, EPI_ADD, false>(a, b, st)));
    }
    if (pn.splits > 1)
      hipLaunchKernelGGL(splitk_finish_kernel<false>, dim3(cdiv((long)nn.M * nn.N / 8, 256)), dim3(256), 0, st,
                         (const float*)scratch, pn.splits, nn.M, nn.N, nn.C, nn.ldc, (const bf16_t*)nullptr, (const bf16_t*)nullptr);
    if (pt.splits > 1)
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3(cdiv((long)tn.M * tn.N / 4, 256)), dim3(256), 0, st,
                         (const float*)partial1, pt.splits, tn.M, tn.N, (float*)tn.C, tn.ldc);
    BM_CHECK_LAUNCH("gemm_joint");
    return BM_OK;
  };
  *rc = launch_all();
  return true;
}

bool gemm_mfma_grouped_supported(int layout, int dtype, int M, int N, int K, int lda, int ldb, int ldc) {
  if (dtype != BM_DTYPE_BF16) return false;
  if (N < 64 || lda % 8 || ldb % 8) return false;
  if (layout == GEMM_TN) return M >= 64 && M % 8 == 0 && N % 8 == 0 && ldc % 4 == 0 && K % MOE_PAD == 0;
  return K >= 64 && K % 8 == 0 && N % 8 == 0 && ldc % 8 == 0 && M % MOE_PAD == 0;
}

bool gemm_mfma_reads_source_rows(int layout, int M, int N, const GemmEpilogue* epi) {
  return layout == GEMM_TN ? M >= 256 && N >= 256 : N >= 256 && epi && (epi->swiglu_fwd_a || epi->swiglu_up);
}

// A row tile is one MOE_PAD block or two of the same group.
bm_status gemm_mfma_grouped(int layout, int M, int N, int K, const void* A, int lda, const void* B,
                            int ldb, void* C, int ldc, const GemmGroups& g, hipStream_t st,
                            const GemmEpilogue* epi) {
  static_assert(MOE_PAD == 128, "the grouped path uses 128-row tiles");
  GemmParams p;
  p.A = (const bf16_t*)A; p.B = (const bf16_t*)B; p.C = C;
  p.bias = nullptr; p.residual = nullptr; p.partial = nullptr;
  p.M = M; p.N = N; p.K = K; p.lda = lda; p.ldb = ldb; p.ldc = ldc;
  p.tiles_m = cdiv(M, 128); p.tiles_n = cdiv(N, 128); p.splits = 1; p.k_per_split = cdiv(K, BK) * BK;
  p.out_fp32 = 0; p.xcd_split = 0;
  p.tile_group = layout == GEMM_TN ? nullptr : g.tile_group;
  p.group_rows = layout == GEMM_TN ? g.group_rows : nullptr;
  p.row_tiles = layout == GEMM_TN ? nullptr : g.row_tiles;
  p.source = g.source; p.src_rows = g.src_rows; p.row_scale = g.row_scale; p.row_dot = g.row_dot;
  if (g.source) {
    // a source row is reached by a 32-bit byte offset from the first one; the rows of a weight gradient's group fit a table in LDS
    const long ld = layout == GEMM_TN && g.source_operand == 1 ? ldb : lda;
    if (!gemm_mfma_reads_source_rows(layout, M, N, epi) || g.src_rows < 1 || g.src_rows * ld * (long)sizeof(bf16_t) > (1L << 32) ||
        (layout == GEMM_TN && g.src_rows > MOE_SOURCE_ROWS)) {
      set_error("grouped gemm: rows of this product are not read from their source");
      return BM_ERR_UNSUPPORTED;
    }
  }
  p.b_group_stride = g.b_stride; p.c_group_stride = g.c_stride;
  p.grid_groups = layout == GEMM_TN ? g.n_groups : 1;
  if (epi) {
    // the SwiGLU epilogues ride on tiles of 256 columns (a tile gathers its weight rows per expert
    // exactly as the dense kernel does per matrix)
    const bool fwd = epi->swiglu_fwd_a != nullptr, bwd = epi->swiglu_up != nullptr;
    if (epi->bias || epi->residual || epi->out_fp32 || fwd == bwd || N % 256 || (fwd && layout != GEMM_NT) ||
        (bwd && (layout != GEMM_NN || !epi->swiglu_dup || !epi->swiglu_a))) {
      set_error("grouped gemm: only the SwiGLU epilogues (forward on NT, backward on NN, N a multiple of 256)");
      return BM_ERR_INVALID_ARG;
    }
    p.sw_up = (const bf16_t*)epi->swiglu_up; p.sw_dup = (bf16_t*)epi->swiglu_dup; p.sw_a = (bf16_t*)epi->swiglu_a;
    p.swf_a = (bf16_t*)epi->swiglu_fwd_a;
  }
  if ((layout == GEMM_TN ? p.group_rows == nullptr || g.n_groups < 1 : p.tile_group == nullptr || p.row_tiles == nullptr)) {
    set_error("grouped gemm: group tables are NULL");
    return BM_ERR_INVALID_ARG;
  }
  if (layout != GEMM_TN && N >= 256) {
    p.tiles_m = g.row_tiles_cap; p.tiles_n = cdiv(N, 256);
    // Walked two at a time, the row tiles of an XCD's CUs belong to half as many experts, of whose weights they read more columns;
    // with more than 8 column tiles two rows of them are more panels than four rows of fewer.  A pass with four and with two, both
    // products up to 2048 columns: 128 experts of 768, 512 rows each 4416 and 4390 us, 768 rows 6057 and 6014, 1024 rows 7485 and 7448, 64 experts
    // of 2048 rows 6790 and 6751; up to 4096 columns: 16 experts of 512 rows 3568 and 3621, 750 rows 4687 and 4717.  With this line none
    // of 18 (8 to 128 experts, 512 to 2048 rows each) is slower than by four or by two.
    p.walk_rows = p.tiles_n <= 8 ? 2 : 4;
    return launch_gemm_alt_groups(layout, p, st);
  }
  if (layout != GEMM_TN) return launch_small(layout, p, st);
  // weight gradient: rows are the contraction index, so the output tile is free; a group's
  // k range is short (a few slices), which makes the per-tile fixed cost count: large tiles
  if (M >= 256 && N >= 256) {
    p.tiles_m = cdiv(M, 256); p.tiles_n = cdiv(N, 256);
    if (g.source) return launch_gemm_alt_tn_source(g.source_operand, p, st);
    return launch_gemm_alt(GEMM_TN, 256, 256, p, st);                     // k ranges are whole slices
  }
  return launch_small(GEMM_TN, p, st);
}

}  // namespace bm
