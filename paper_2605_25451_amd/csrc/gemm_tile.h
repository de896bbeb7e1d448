// Shared by the bf16 matrix-core GEMM kernels: the launch parameters, the map from workgroup to tile,
// the fragment types and the epilogue.
#pragma once
#include "common.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace bm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int BK = 64;          // k slice
constexpr int KCH = BK / 8;     // 16-byte chunks per k-contiguous row

struct GemmParams {
  const bf16_t* A; const bf16_t* B; void* C;
  const bf16_t* bias; const bf16_t* residual;
  const bf16_t* sw_up = nullptr; bf16_t* sw_dup = nullptr; bf16_t* sw_a = nullptr;   // SwiGLU backward epilogue (see GemmEpilogue)
  bf16_t* swf_a = nullptr;      // SwiGLU forward epilogue (see GemmEpilogue); N = 2F
  float* partial;               // splits > 1: fp32 partial tiles [split][M][N]
  int M, N, K, lda, ldb, ldc;
  int tiles_m, tiles_n, splits, k_per_split;
  int out_fp32;
  int xcd_split;                // each k split owns 8/splits XCDs (splits in {2,4,8})
  // grouped problems (see GemmGroups); all null / zero otherwise
  const int32_t* tile_group;
  const int32_t* group_rows;
  const int32_t* row_tiles;
  long b_group_stride, c_group_stride;
  // rows read where they lie instead of from a sorted copy: the source row (of src_rows) of each row of A (grouped NT and NN) or of
  // each k row of one operand (grouped TN); what is out of range reads the first row of its tile or group
  const int32_t* source; int src_rows;
  const float* row_scale;       // SwiGLU backward: a factor of every row of the product ...
  float* row_dot;               // ... and [rows, N / 64]: the product times the activation, both without it, summed over 64 columns
  int big_rows;                 // of launch_gemm_alt_mixed: rows of 256x256 tiles, before tiles_m - big_rows of 128x256
  int walk_rows;                // of launch_gemm_alt_groups: row tiles that are walked side by side, 2 or 4
  int grid_groups;              // host: workgroups = tiles * splits * grid_groups (>= 1)
};

// Weight gradients that share a grid: the parts' workgroups lie behind one another, first those of parts with one k range.
struct TnParts {
  static constexpr int MAX = 4;
  struct Part {
    const bf16_t *A, *B; float *C, *partial;
    int M, N, K, lda, ldb, ldc, tiles_m, tiles_n, splits, k_per_split, xcd_split, first_wg;
  } part[MAX];
  int n, one_list;              // one_list: workgroups of the parts with one k range, if their tiles lie in one list
  int wgs() const { const Part& l = part[n - 1]; return l.first_wg + l.tiles_m * l.tiles_n * l.splits; }
};

// acc += a b^T with v_mfma_f32_16x16x32_bf16.  Written as an asm statement that ties the
// accumulator block to the accumulation half of the register file: the allocator otherwise keeps
// some blocks in the other half, with copies between the halves inside the loop.  The compiler
// does not know that the statement is an MFMA; what keeps the accumulators safe is that a block is next
// touched 16 MFMAs later, as the accumulator of the same instruction again, which asks for no wait
// state at any distance, and that gemm_epilogue() waits before it reads them.
__device__ inline void mfma16(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// acc = a b^T: the first product of a tile takes the constant 0 as its addend, so the accumulators
// are never initialised by separate instructions (which the compiler, not knowing that the asm
// statement is an MFMA, would place right in front of it without the wait states that needs)
__device__ inline void mfma16_first(f32x4& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(acc) : "v"(a), "v"(b));
}

// f(0), f(1), ..., f(N-1) with the index as a compile-time constant
template <int N, int I = 0, typename F>
__device__ inline void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<N, I + 1>(f);
  }
}

// XCD-aware tile order: workgroup ids go round-robin over the 8 XCDs, so give each XCD a contiguous run of the tiles (the
// first total % 8 of them one tile more), walked in column-major groups of GROUP_M tile rows (operand reuse in that XCD's L2).
__device__ inline int xcd_run(int pid, int total) {
  const int xcd = pid % 8;
  return xcd * (total / 8) + min(xcd, total % 8) + pid / 8;
}
template <int GROUP_M>
__device__ inline void grouped_tile(int id, int tiles_m, int tiles_n, int* tm, int* tn) {
  const int per_group = GROUP_M * tiles_n;
  const int g = id / per_group;
  const int first_m = g * GROUP_M;
  const int gsize = min(tiles_m - first_m, GROUP_M);
  const int in = id % per_group;
  *tm = first_m + in % gsize;
  *tn = in / gsize;
}

// K split with XCD affinity: split s owns the 8/splits XCDs s*G .. s*G+G-1 and each of
// them a contiguous run of that split's tiles, so an operand panel of one k range is
// fetched by as few L2s as possible (HBM traffic of the weight gradient is dominated by
// panels fetched once per XCD that touches them).
__device__ inline void split_tile_of_block(int pid, int tiles, int splits, int tiles_m, int tiles_n,
                                           int* split, int* tm, int* tn) {
  const int G = 8 / splits;
  const int xcd = pid & 7, local = pid >> 3;
  *split = xcd / G;
  grouped_tile<8>((xcd % G) * (tiles / G) + local, tiles_m, tiles_n, tm, tn);
}

__device__ inline void tile_of_block(int pid, int total, int tiles_m, int tiles_n, int* tm, int* tn) {
  grouped_tile<4>(xcd_run(pid, total), tiles_m, tiles_n, tm, tn);     // measured: 4 tile rows per group is a little ahead of 8, 2 and 16
}

// What the epilogue does with the product, fixed at compile time: one straight run of instructions
// per kind (with run-time switches between the strips the K = 1024 products lost 5 %).
enum { EPI_PLAIN = 0,     // C = acc (+bias), bf16 or fp32
       EPI_RES,           // C = acc (+bias) + residual
       EPI_SWIGLU_FWD, EPI_SWIGLU_BWD,
       EPI_ADD,           // fp32 C += acc
       EPI_PARTIAL };     // acc -> this split's partial tile


// Where a workgroup's tile lies: operands (B of the tile's group), first row and column, k range.
// kbeg == kend: nothing to do.
// All values are workgroup-uniform.
struct TileJob {
  const bf16_t *A, *B;
  int m0, n0, tn, kbeg, kend, split;
  long c_off;
};

template <int BM, int BN>
__device__ inline TileJob tile_job(const GemmParams& p, int split, int tm, int tn) {
  TileJob t;
  t.split = split; t.tn = tn;
  t.m0 = tm * BM; t.n0 = t.tn * BN;
  t.kbeg = t.split * p.k_per_split;
  t.kend = min(p.K, t.kbeg + p.k_per_split);
  t.A = p.A; t.B = p.B;
  t.c_off = 0;
  if (p.group_rows) {
    // grouped weight gradient: `split` is the group; its rows are the k range
    t.kbeg = min(p.group_rows[t.split], p.K);
    t.kend = max(t.kbeg, min(p.group_rows[t.split + 1], p.K));
    t.c_off = (long)t.split * p.c_group_stride;
    t.split = 0;
  } else if (p.tile_group) {
    const int g = p.tile_group[t.m0 / MOE_PAD];
    if (g < 0) t.kend = t.kbeg;
    else t.B += (long)g * p.b_group_stride;
  }
  return t;
}

template <int BM, int BN>
__device__ inline TileJob locate_tile(const GemmParams& p, int pid) {
  const int tiles = p.tiles_m * p.tiles_n;
  int split = pid / tiles, tm, tn;
  if (p.xcd_split) split_tile_of_block(pid, tiles, p.splits, p.tiles_m, p.tiles_n, &split, &tm, &tn);
  else tile_of_block(pid % tiles, tiles, p.tiles_m, p.tiles_n, &tm, &tn);
  return tile_job<BM, BN>(p, split, tm, tn);
}

// The accumulators behind the last MFMAs, readable: the compiler does not know that the asm statements are MFMAs and
// leaves no wait states between them and what reads their results, and arithmetic on the results (a conversion, a copy to
// the other half of the register file) may move in front of the wait unless it depends on it.
template <int FM, int FN>
__device__ inline void settle(f32x4 (&acc)[FM][FN]) {
  asm volatile("s_nop 15\n\ts_nop 15");
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) asm volatile("" : "+a"(acc[i][j]));
  __builtin_amdgcn_sched_barrier(0);
}

template <int FN> constexpr int epilogue_stage_floats() { return 2 * 16 * (FN * 16 + 4); }

// fp32 outputs of weight gradients and k ranges (EPI_ADD, EPI_PARTIAL): 4 columns per lane, so that a load or store
// instruction covers 4 rows of 256 contiguous bytes (with 8 columns per lane every instruction touched half of each
// 32 bytes and the caches took twice the requests); two strips of LDS in turn; the old C four strips ahead, the last two
// of them once the fragments are dead.  The epilogue of a lone 256x256 tile, until its last store is issued, 6.0 -> 4.2 us, with all CUs at
// work 16-19 -> 15-18; 22016x4096 over 8192 rows 1152 -> 1109 us, over 777 241 -> 235, 4096x11008 over 777 134 -> 128.
// One lane offset serves all rows of a tile that lies inside C: with an address per row the ragged and the full path
// together spill.
template <int EPI, int FM, int FN, typename RowOf, typename Last>
__device__ inline void gemm_epilogue_f32(const GemmParams& p, f32x4 (&acc)[FM][FN], float* stage, int lane, int col0,
                                         int split, long c_off, bool full, RowOf row_of, Last last) {
  constexpr int SLD = FN * 16 + 4;
  constexpr int LPR = FN * 4, RPI = 64 / LPR, TPS = 16 / RPI;
  constexpr int AHEAD = 4;
  const int m_in = lane & 15, q4 = (lane >> 4) * 4;
  const int rcol = (lane % LPR) * 4, rrow = lane / LPR;
  const int gn = col0 + rcol;
  // a tile that lies inside C: one lane offset for all its rows, the rest of an address is uniform
  const uint32_t lane_off = ((uint32_t)rrow * (uint32_t)p.ldc + (uint32_t)rcol) * 4u;
  const float* c_base = (const float*)p.C + c_off + col0;
  f32x4 pre[AHEAD][TPS];
  auto request = [&](auto i_t, bool inside) {
    constexpr int i = decltype(i_t)::value;
    if (EPI != EPI_ADD || i >= FM) return;
#pragma unroll
    for (int t = 0; t < TPS; ++t) {
      const char* at;
      if (inside) {
        at = reinterpret_cast<const char*>(c_base + (size_t)(row_of(i) + t * RPI) * p.ldc) + lane_off;
      } else {
        const int gm = min(row_of(i) + t * RPI + rrow, p.M - 1), gc = min(gn, p.N - 4);
        at = reinterpret_cast<const char*>((const float*)p.C + c_off + (size_t)gm * p.ldc + gc);
      }
      pre[i % AHEAD][t] = *reinterpret_cast<const f32x4*>(at);
    }
  };
  request(std::integral_constant<int, 0>{}, full);
  request(std::integral_constant<int, 1>{}, full);
  last();
  settle(acc);
  auto finish = [&](auto full_t, auto strips_t) {
    constexpr bool FULL = decltype(full_t)::value;
    constexpr int STRIPS = decltype(strips_t)::value;
    static_for<AHEAD - 2>([&](auto i_t) {
      if (decltype(i_t)::value + 2 < STRIPS) request(std::integral_constant<int, decltype(i_t)::value + 2>{}, FULL);
    });
    static_for<STRIPS>([&](auto i_t) {
      constexpr int i = decltype(i_t)::value;
      float* strip = stage + (i & 1) * (16 * SLD);
#pragma unroll
      for (int j = 0; j < FN; ++j) *reinterpret_cast<f32x4*>(strip + m_in * SLD + j * 16 + q4) = acc[i][j];
#pragma unroll
      for (int t = 0; t < TPS; ++t) {
        const int row = t * RPI + rrow, gm = row_of(i) + row;
        f32x4 out = *reinterpret_cast<const f32x4*>(strip + row * SLD + rcol);
        if (EPI == EPI_ADD) out += pre[i % AHEAD][t];
        if (!FULL && !(gm < p.M && gn < p.N)) continue;
        if (EPI == EPI_PARTIAL)
          *reinterpret_cast<f32x4*>(p.partial + ((size_t)split * p.M + gm) * p.N + gn) = out;
        else if (FULL)
          *reinterpret_cast<f32x4*>(reinterpret_cast<char*>(const_cast<float*>(c_base) + (size_t)(row_of(i) + t * RPI) * p.ldc) +
                                    lane_off) = out;
        else
          *reinterpret_cast<f32x4*>((float*)p.C + c_off + (size_t)gm * p.ldc + gn) = out;
      }
      if (i + AHEAD < STRIPS) request(std::integral_constant<int, i + AHEAD>{}, FULL);
    });
  };
  // Partial tiles of few rows (decoding): wavefronts past them store nothing, others one strip.  4 rows x 280 x 5160, NN, 14 k ranges: all
  // strips 12.6 us, this 12.2; 128 x 80 x 7475, TN, 24 ranges, 15.1 -> 14.1.  (A test in front of every strip keeps them from overlapping:
  // 64 x 64 x 4000, TN, 12.0 -> 13.2; the same for EPI_ADD: a block of 1000 rows 289.0 -> 290.4.)
  if (full) {
    finish(std::true_type{}, std::integral_constant<int, FM>{});
  } else if (EPI != EPI_PARTIAL) {
    finish(std::false_type{}, std::integral_constant<int, FM>{});
  } else if (row_of(0) < p.M && col0 < p.N) {
    if (row_of(1) < p.M) finish(std::false_type{}, std::integral_constant<int, FM>{});
    else finish(std::false_type{}, std::integral_constant<int, 1>{});
  }
}

// ---- epilogue of one wavefront: FM x FN accumulator blocks of 16x16.  The MFMAs run with swapped
// operands, so block (i,j) holds C^T: lane = row m = l%16, registers = 4 consecutive columns
// n = 4*(l/16) + e.  Each wavefront transposes its own 16-row strips through LDS and then writes
// whole rows, 16 bytes per lane (fp32 outputs: above).
//
// What the epilogue combines with the product -- the residual, the saved g and u of the SwiGLU
// backward -- is requested two strips ahead (the old C of a weight gradient four), the first two strips before
// the tile's last MFMAs (`last`): fetched in front of each store instead, a tile pays one memory
// latency per store instruction, 32 of them in a row (four wavefronts of 128x128, the old C: dW 22016x4096
// over 777 rows 296 -> 247 us, over 8192 rows 1301 -> 1271 us).  Addresses are clamped into the matrix, so
// that the requests carry no condition.
//   row_of(i)   first row of strip i;  col0  the wavefront's first column
//   acol0       SwiGLU forward: its first column of a
//   stage       epilogue_stage_floats() of LDS of its own; free to write once `last` has returned
//   full        the tile lies inside C, so no store carries a condition (a conditional store makes the
//               wait for the next strip's operands wait for the stores as well)
template <int EPI, int FM, int FN, typename RowOf, typename Last>
__device__ inline void gemm_epilogue(const GemmParams& p, f32x4 (&acc)[FM][FN], float* stage, int lane, int col0,
                                     int acol0, int split, long c_off, bool full, RowOf row_of, Last last) {
  if constexpr (EPI == EPI_ADD || EPI == EPI_PARTIAL) {
    gemm_epilogue_f32<EPI>(p, acc, stage, lane, col0, split, c_off, full, row_of, last);
    return;
  }
  constexpr int TN_ = FN * 16;
  constexpr int SLD = TN_ + 4;                          // padded fp32 row: conflict-free both ways
  constexpr int LPR = TN_ / 8;                          // lanes per output row (8 columns each)
  constexpr int RPI = 64 / LPR;                         // rows per store instruction
  constexpr int TPS = 16 / RPI;                         // store instructions per strip
  static_assert(16 % RPI == 0, "a 16-row strip must be a whole number of store instructions");
  const int m_in = lane & 15, q4 = (lane >> 4) * 4;
  const int rcol = (lane % LPR) * 8, rrow = lane / LPR;
  const int gn = col0 + rcol;
  u32x4 pre[2][TPS][2];
  float scale[2][TPS];
  auto request = [&](auto i_t) {
    constexpr int i = decltype(i_t)::value;
    if (i >= FM) return;
#pragma unroll
    for (int t = 0; t < TPS; ++t) {
      const int gm = min(row_of(i) + t * RPI + rrow, p.M - 1), gc = min(gn, p.N - 8);
      if (EPI == EPI_SWIGLU_BWD) {
        const bf16_t* up = p.sw_up + (size_t)gm * (2 * p.N) + gc;
        pre[i & 1][t][0] = *reinterpret_cast<const u32x4*>(up);
        pre[i & 1][t][1] = *reinterpret_cast<const u32x4*>(up + p.N);
        scale[i & 1][t] = p.row_scale ? p.row_scale[gm] : 1.f;
      } else if (EPI == EPI_RES) {
        pre[i & 1][t][0] = *reinterpret_cast<const u32x4*>(p.residual + (size_t)gm * p.ldc + gc);
      }
    }
  };
  request(std::integral_constant<int, 0>{});
  request(std::integral_constant<int, 1>{});
  last();
  settle(acc);

  float bias[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) bias[e] = 0.f;
  if ((EPI == EPI_PLAIN || EPI == EPI_RES) && p.bias && gn < p.N) load16(p.bias + gn, bias);
  auto finish = [&](auto full_t) {
    constexpr bool FULL = decltype(full_t)::value;
    static_for<FM>([&](auto i_t) {
      constexpr int i = decltype(i_t)::value;
#pragma unroll
      for (int j = 0; j < FN; ++j)
        *reinterpret_cast<f32x4*>(stage + m_in * SLD + j * 16 + q4) = acc[i][j];
      if (EPI == EPI_SWIGLU_FWD) {
        // SwiGLU forward: the strip holds g in its first TN_/2 columns and u in the others, of the
        // same TN_/2 columns of a; a lane takes 8 of them
        constexpr int HW = TN_ / 2, LPR2 = HW / 8, RPI2 = 64 / LPR2;
        const int F = p.N / 2;
        const int rcol2 = (lane % LPR2) * 8, rrow2 = lane / LPR2;
        const int acol = acol0 + rcol2;
#pragma unroll
        for (int t = 0; t < (16 + RPI2 - 1) / RPI2; ++t) {
          const int row = t * RPI2 + rrow2;
          const int gm = row_of(i) + row;
          if (row < 16 && gm < p.M) {
            const f32x4 g0 = *reinterpret_cast<const f32x4*>(stage + row * SLD + rcol2);
            const f32x4 g1 = *reinterpret_cast<const f32x4*>(stage + row * SLD + rcol2 + 4);
            const f32x4 u0 = *reinterpret_cast<const f32x4*>(stage + row * SLD + HW + rcol2);
            const f32x4 u1 = *reinterpret_cast<const f32x4*>(stage + row * SLD + HW + rcol2 + 4);
            union { u32x4 v; bf16_t h[8]; } pg, pu, pa;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              pg.h[e] = Elt<bf16_t>::from_f(e < 4 ? g0[e] : g1[e - 4]);
              pu.h[e] = Elt<bf16_t>::from_f(e < 4 ? u0[e] : u1[e - 4]);
              const float g = (float)pg.h[e], u = (float)pu.h[e];
              const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
              pa.h[e] = Elt<bf16_t>::from_f(g * sig * u);
            }
            bf16_t* c = (bf16_t*)p.C + (size_t)gm * p.ldc + acol;
            __builtin_nontemporal_store(pg.v, reinterpret_cast<u32x4*>(c));
            __builtin_nontemporal_store(pu.v, reinterpret_cast<u32x4*>(c + F));
            *reinterpret_cast<u32x4*>(p.swf_a + (size_t)gm * F + acol) = pa.v;
          }
        }
        return;
      }
#pragma unroll
      for (int t = 0; t < TPS; ++t) {
        const int row = t * RPI + rrow;
        const int gm = row_of(i) + row;
        const f32x4 lo = *reinterpret_cast<const f32x4*>(stage + row * SLD + rcol);
        const f32x4 hi = *reinterpret_cast<const f32x4*>(stage + row * SLD + rcol + 4);
        if (!FULL && !(gm < p.M && gn < p.N)) continue;
        float out[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        const size_t idx = (size_t)gm * p.ldc + gn;
        if (EPI == EPI_SWIGLU_BWD) {
          // out = dA of 8 columns of one row: d_up and the activation instead of C
          const size_t up_idx = (size_t)gm * (2 * p.N) + gn;
          union { u32x4 u; bf16_t h[8]; } sg{pre[i & 1][t][0]}, su{pre[i & 1][t][1]};
          float dg[8], du[8], av[8];
          const float sc = scale[i & 1][t];                    // on the activation as well: it is only read for the weight gradient
          float dot = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float g = (float)sg.h[e], u = (float)su.h[e];
            const float sig = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * g));
            dot += out[e] * (g * sig * u);
            const float sl = sc * (g * sig);                   // silu(g)
            av[e] = sl * u;
            du[e] = out[e] * sl;
            dg[e] = sc * out[e] * u * sig * (1.0f + g * (1.0f - sig));
          }
          if (p.row_dot) {
#pragma unroll
            for (int off = 1; off < LPR; off <<= 1) dot += __shfl_xor(dot, off, WAVE);
            if (lane % LPR == 0) p.row_dot[(size_t)gm * (p.N / TN_) + col0 / TN_] = dot;
          }
          store16(p.sw_dup + up_idx, dg);
          store16(p.sw_dup + up_idx + p.N, du);
          store16(p.sw_a + (size_t)gm * p.N + gn, av);
          continue;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] += bias[e];
        if (EPI == EPI_RES) {
          union { u32x4 u; bf16_t h[8]; } r{pre[i & 1][t][0]};
#pragma unroll
          for (int e = 0; e < 8; ++e) out[e] += (float)r.h[e];
        }
        if (p.out_fp32) {
          float* c = (float*)p.C + idx;
          *reinterpret_cast<f32x4*>(c) = f32x4{out[0], out[1], out[2], out[3]};
          *reinterpret_cast<f32x4*>(c + 4) = f32x4{out[4], out[5], out[6], out[7]};
        } else {
          union { u32x4 u; bf16_t h[8]; } pk;
#pragma unroll
          for (int e = 0; e < 8; ++e) pk.h[e] = Elt<bf16_t>::from_f(out[e]);
          __builtin_nontemporal_store(pk.u, reinterpret_cast<u32x4*>((bf16_t*)p.C + idx));
        }
      }
      request(std::integral_constant<int, i + 2>{});
    });
  };
  constexpr bool FETCHES = EPI == EPI_RES || EPI == EPI_SWIGLU_BWD;
  if (FETCHES && full) finish(std::true_type{});
  else finish(std::false_type{});
}

// gemm_alt.hip: the tile (256x256, 128x256 or 256x128) of a plan
bm_status launch_gemm_alt(int layout, int bm, int bn, const GemmParams& p, hipStream_t st);
// NT and NN: the first big_rows x 256 rows on 256x256 tiles, the others on 128x256
bm_status launch_gemm_alt_mixed(int layout, const GemmParams& p, hipStream_t st);
// grouped NT and NN on the row tiles that p lists; tiles_m: their capacity
bm_status launch_gemm_alt_groups(int layout, const GemmParams& p, hipStream_t st);
// grouped weight gradients whose A (operand 0) or B (1) is read from its source rows; no group longer than MOE_SOURCE_ROWS
bm_status launch_gemm_alt_tn_source(int operand, const GemmParams& p, hipStream_t st);
// weight gradients in one grid of 256x256 tiles
bm_status launch_gemm_alt_tn_parts(const TnParts& g, hipStream_t st);

}  // namespace bm
