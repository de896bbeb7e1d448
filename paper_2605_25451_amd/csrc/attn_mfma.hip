// Variable-length flash attention on the gfx950 matrix cores (bf16 in, fp32
// accumulate, online softmax in base 2), forward and backward.
//
// Packing: a workgroup owns one tile of 128 or 256 rows of ONE sequence and one head, so
// attention is block-diagonal by construction; tiles are enumerated by walking
// cu_seqlens (no padded grid), longest-running tiles first.
//
// Layout trick.  All score matrices are produced TRANSPOSED by the MFMA
// (keys x queries for forward/dQ, queries x keys for dK/dV), so that the
// softmax statistic of a row lives in ONE lane (two lanes for the two 32-lane
// halves) instead of being spread over a wavefront, and the fp32 accumulator
// of one MFMA is -- after conversion to bf16 -- exactly the B operand of the
// next MFMA (P feeds P*V, dS feeds dS*K / dS*Q): probabilities never touch LDS.
// The matching A operands (V^T, K^T, Q^T, dO^T) come from the LDS transpose
// read (ds_read_b64_tr_b16) of tiles stored in their natural [row][dh] form.
// Tiles are XOR-swizzled with a pattern that is conflict-free for both the
// 16-byte row reads and the transpose reads.
//
// Backward is split in two kernels (dK/dV per key tile, dQ per query tile),
// each recomputing P from the saved log-sum-exp: every output element has one
// owner, so there are no floating-point atomics and results are reproducible.
#include "common.h"

#include <type_traits>

namespace bm {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// Head sizes: 64 and 128 fit the 32x32x16 MFMA exactly; 72 (the DiT blocks) is run
// with its contraction padded to 80 and its output rows padded to 96 by zero chunks
// that exist only in LDS and registers, never in HBM.
template <int DH>
struct HeadDim {
  static constexpr int KS = (DH + 15) / 16;    // k=16 steps when dh is the contraction index
  static constexpr int NB = (DH + 31) / 32;    // 32-row blocks when dh is an output index
  static constexpr int DHL = NB * 32;          // LDS row width in elements
  static constexpr int VCH = DH / 8;           // 16-byte chunks of a row that hold data
};

// ---- swizzled [rows][DHL] bf16 tile -----------------------------------------
template <int DHL>
__device__ inline int tile_swizzle(int row) {      // chunk c of a row sits in slot c ^ tile_swizzle(row)
  if (DHL == 128) return ((row & 3) << 2) | ((row >> 2) & 3);
  if (DHL == 96) return (row >> 2) & 3;
  const int v = row >> 1;
  return ((v & 1) << 2) | ((v >> 1) & 3);
}
template <int DHL>
__device__ inline int tile_off(int row, int c) {   // element offset of 16-byte chunk c of a row
  return row * DHL + ((c ^ tile_swizzle<DHL>(row)) << 3);
}

// 8 consecutive dh values (chunk c) of a global row as an MFMA operand; zeros past dh
template <int DH>
__device__ inline bf16x8 load_chunk(const bf16_t* row, int c) {
  if (DH % 16 == 0 || c < HeadDim<DH>::VCH) return *reinterpret_cast<const bf16x8*>(row + c * 8);
  bf16x8 z;
#pragma unroll
  for (int e = 0; e < 8; ++e) z[e] = (bf16_t)0.f;
  return z;
}

// operand fragment, rows of the tile are the MFMA row/col index, dh is the k index:
// lane l -> tile row row0 + l%32, dh = ks*16 + (l/32)*8 .. +7
template <int DH>
__device__ inline bf16x8 frag_rows(const bf16_t* t, int row0, int ks, int lane) {
  return *reinterpret_cast<const bf16x8*>(t + tile_off<DH>(row0 + (lane & 31), ks * 2 + (lane >> 5)));
}

// A operand X^T: MFMA row = dh index col0 + l%32, k index = tile rows, in the
// order the fp32 accumulator of a transposed score block hands them over:
// half h = l/32 supplies tile rows r0+4h..+3 and r0+8+4h..+3.
template <int DH>
__device__ inline bf16x8 frag_cols(const bf16_t* t, int col0, int r0, int lane) {
  const int gi = lane >> 4, s = lane & 15;
  const int col = col0 + (gi & 1) * 16 + (s & 3) * 4;
  const int row = r0 + (gi >> 1) * 4 + (s >> 2);
  const bf16_t* p0 = t + tile_off<DH>(row, col >> 3) + (col & 7);
  const bf16_t* p1 = t + tile_off<DH>(row + 8, col >> 3) + (col & 7);
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p0);
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p1);
  union { struct { s16x4 a, b; } s; bf16x8 v; } u;
  u.s.a = lo; u.s.b = hi;
  return u.v;
}

// max / sum of a value with the one held by the lane 32 away (the two halves of a wavefront own
// the same score column): v_permlane32_swap exchanges the halves in the vector unit, without the
// trip through the LDS crossbar that a lane shuffle takes
__device__ inline float max_with_other_half(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ inline float sum_with_other_half(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// accumulator rows 8t..8t+7 of a 32x32 block -> bf16 B operand of a k=16 step
__device__ inline bf16x8 acc_to_operand(const f32x16& a, int t) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = (bf16_t)a[t * 8 + e];
  return r;
}

// ---- global -> LDS: a [ROWS][DH] tile brought in by NT threads -------------------
// 16-byte loads that write LDS directly (no registers, no LDS store
// instructions): lane l of a wavefront fills bytes [16 l, 16 l + 16) of a 1 KiB run of slots, so the
// swizzle is applied on the global side -- the lane that owns slot s of a row fetches chunk
// s ^ tile_swizzle(row).  Padding slots (head sizes that are no multiple of 32) are never written
// by a load: zero() clears them once.  The loads are asynchronous: wait for vmcnt(0), then a
// workgroup barrier, before any wavefront reads the tile.
template <int ROWS, int DH, int NT>
struct TileAsync {
  static constexpr int DHL = HeadDim<DH>::DHL;
  static constexpr int CPR = DHL / 8;
  static constexpr int SLOTS = ROWS * CPR;
  static constexpr int CH = (SLOTS + NT - 1) / NT;    // loads per thread (the last round may be short)
  // UNI: every load of a thread has the same chunk, and rows a fixed distance apart
  static constexpr bool UNI = NT % CPR == 0 && (NT / CPR) % 16 == 0 && SLOTS % NT == 0;
  static constexpr int RSTEP = NT / CPR, NV = UNI ? 1 : CH;
  static_assert(SLOTS % 64 == 0 && NT % 64 == 0, "a tile is a whole number of 1 KiB runs");
  static constexpr bool ALL_LIVE = DHL == DH && SLOTS % NT == 0;   // no padding slot, no short round
  uint32_t goff[NV];    // byte offset of a load from the tile's first row (full tiles)
  int tid_;             // the thread's index among the NT that bring the tile in
  // (row, chunk) of load i; false: it would fill a padding slot or lies past the tile
  __device__ inline bool place(int i, int* row, int* chunk, int tid) const {
    const int id = tid + i * NT;
    *row = id / CPR;
    *chunk = (id % CPR) ^ tile_swizzle<DHL>(*row);
    return ALL_LIVE || (id < SLOTS && *chunk < HeadDim<DH>::VCH);
  }
  __device__ inline void init(int ld, int tid) {
    tid_ = tid;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      int row, c;
      place(i, &row, &c, tid);
      goff[i] = (uint32_t)row * (uint32_t)ld * 2u + (uint32_t)c * 16u;
    }
  }
  // One 16-byte load per lane straight into LDS.  Written as inline assembly so that the compiler does
  // not see an LDS write in flight: it would otherwise make every LDS read that follows wait for
  // vmcnt(0) and the tile would no longer stream in behind the arithmetic.  The caller orders the
  // reads of a tile after wait_async_tiles() and a barrier.
  static __device__ inline void load16(const void* base, uint32_t voff, uint32_t lds_addr) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0");
  }
  // base: first row of the tile (wave-uniform); rows_left: valid rows from there (>= 1), rows beyond
  // them are clamped to the last valid one (their results are masked or unused); wave: wave-uniform
  __device__ inline void issue(const bf16_t* __restrict__ base_in, int ld, int rows_left, bf16_t* t,
                               int wave) const {
    // the base goes into the asm statement as a scalar register pair: say so, wherever the caller's
    // arithmetic left it
    const uint64_t b64 = reinterpret_cast<uint64_t>(base_in);
    const bf16_t* base = reinterpret_cast<const bf16_t*>(
        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b64 >> 32)) << 32) |
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b64));
    rows_left = __builtin_amdgcn_readfirstlane(rows_left);
    const uint32_t dst = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)(t + wave * 512);
    if (rows_left >= ROWS) {
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        int row, c;
        // (UNI: the distance between a thread's loads goes into the scalar base, not into a register each)
        if (place(i, &row, &c, tid_))
          load16(base + (UNI ? (size_t)(i * RSTEP) * ld : (size_t)0), goff[UNI ? 0 : i], dst + i * NT * 16);
      }
    } else {
      // a cut tile (the last one of a sequence): offsets from scratch, rows clamped.  The thread index
      // passes through an empty asm so that none of this is computed ahead of the loop and kept in
      // registers for the one step that needs it.
      int t_op = tid_;
      asm volatile("" : "+v"(t_op));
#pragma unroll
      for (int i = 0; i < CH; ++i) {
        int row, c;
        if (place(i, &row, &c, t_op))
          load16(base, (uint32_t)min(row, rows_left - 1) * (uint32_t)ld * 2u + (uint32_t)c * 16u, dst + i * NT * 16);
      }
    }
  }
  static __device__ inline void zero_padding(bf16_t* t, int tid) {
    if (DHL == DH) return;
#pragma unroll
    for (int i = 0; i < CH; ++i) {
      const int id = tid + i * NT;
      const int r = id / CPR, c = (id % CPR) ^ tile_swizzle<DHL>(r);
      if (id < SLOTS && c >= HeadDim<DH>::VCH) *reinterpret_cast<u32x4*>(t + id * 8) = u32x4{0u, 0u, 0u, 0u};
    }
  }
};
// The tile loads are invisible to the compiler's wait-count bookkeeping, so the wait for them is
// written out as well.  A vmcnt wait that the compiler adds for one of ITS loads would also wait for
// tile loads in flight: settle_compiler_loads() (a wait the bookkeeping does read) goes once in front
// of a loop that streams tiles, after the kernel's ordinary loads, so that none is added inside.
__device__ inline void wait_async_tiles() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
__device__ inline void settle_compiler_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); /* vmcnt(0) */ }

// The order in which the tiles of the sequences are handed out: workgroups are dispatched in id
// order, so the sequences whose tiles run longest go first and the short ones fill the tail of the
// launch.  Built on the host from the host copy of the offsets (the same copy that sizes the grid)
// and passed by value in the kernel arguments: nothing to allocate or copy, and a workgroup finds
// its tile from one batch of scalar loads instead of a dependent load per sequence.  Any order
// gives the same results, only the schedule changes.  n == 0: no table (more than 64 sequences),
// the kernel walks the offsets in pack order.
struct SeqOrder {
  int n;                // positions in use, a multiple of 16
  uint32_t w[64];       // position i: sequence index in bits 0..7, its number of tiles above
};

// cu_tiles: offsets of the side that is cut into tiles of `rows` rows; cu_cost: offsets of the side
// a tile loops over (its running time).  sorted = false keeps the pack order: under a causal mask
// a pack has tiles of every length whatever the order, and the long sequences' tiles all running at
// once measured slower (their operands no longer fit the L2 of an XCD together).
SeqOrder make_seq_order(const int32_t* cu_tiles, const int32_t* cu_cost, int S, int rows, bool sorted) {
  SeqOrder o;
  o.n = 0;
  for (int i = 0; i < 64; ++i) o.w[i] = 0;          // unused positions: sequence 0, no tile
  if (S < 1 || S > 64) return o;
  for (int s = 0; s < S; ++s)
    if ((cu_tiles[s + 1] - cu_tiles[s] + rows - 1) / rows >= (1 << 24)) return o;
  unsigned char idx[64];
  for (int i = 0; i < S; ++i) idx[i] = (unsigned char)i;
  // stable insertion sort by descending length
  for (int i = 1; sorted && i < S; ++i) {
    const unsigned char x = idx[i];
    const int lx = cu_cost[x + 1] - cu_cost[x];
    int j = i;
    while (j > 0 && cu_cost[idx[j - 1] + 1] - cu_cost[idx[j - 1]] < lx) { idx[j] = idx[j - 1]; --j; }
    idx[j] = x;
  }
  o.n = (S + 15) / 16 * 16;
  for (int i = 0; i < S; ++i) {
    const int nt = (cu_tiles[idx[i] + 1] - cu_tiles[idx[i]] + rows - 1) / rows;
    o.w[i] = ((uint32_t)nt << 8) | idx[i];
  }
  return o;
}

// which (sequence, tile) a linear tile id is; tiles of `rows` rows, later tiles of a
// sequence first (under a causal mask they are the long ones).  Wave-uniform throughout.
__device__ inline bool find_tile(const int32_t* __restrict__ cu, const SeqOrder& ord, int S, int rows, int id,
                                 int* seq, int* tile, int* ntiles) {
  if (ord.n == 0) {
    for (int s = 0; s < S; ++s) {
      const int L = cu[s + 1] - cu[s];
      const int nt = (L + rows - 1) / rows;
      if (id < nt) { *seq = s; *tile = nt - 1 - id; *ntiles = nt; return true; }
      id -= nt;
    }
    return false;
  }
  for (int s0 = 0; s0 < ord.n; s0 += 16) {
    uint32_t e[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) e[j] = ord.w[s0 + j];
    int found = -1, fid = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {               // branch-free choice among the sixteen
      const int n = (int)(e[j] >> 8);
      const bool here = found < 0 && id < n;
      found = here ? (int)e[j] : found;
      fid = here ? id : fid;
      id -= found < 0 ? n : 0;
    }
    if (found >= 0) {
      const int nt = found >> 8;
      *seq = found & 255; *tile = nt - 1 - fid; *ntiles = nt;
      return true;
    }
  }
  return false;
}

// Linear workgroup id -> (tile id, head).  Heads vary fastest, and since workgroup
// ids go round-robin over the 8 XCDs, head index i lands on XCD i%8: give XCD x
// the consecutive heads x*(H/8).., so every tile of one head -- and the q heads of
// one GQA group -- meet their K/V in the same XCD's L2.
__device__ inline void tile_and_head(int H, int* tile, int* head, int b) {
  const int i = b % H;
  *tile = b / H;
  *head = (H % 8 == 0) ? (i % 8) * (H / 8) + i / 8 : i;
}

// =============================================================================
// forward
// =============================================================================
constexpr int NUM_CU = 256;
constexpr int FQ = 128;   // query rows per workgroup (32 per wavefront)
constexpr int FK = 64;    // keys per step

template <int DH, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void fa_fwd_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk, int S,
    bf16_t* __restrict__ o, int ldo, float* __restrict__ lse, int Ttot, int Hq, int group,
    float scale_log2, SeqOrder ord) {
  // K and V tiles are double-buffered: tile kt+1 streams into LDS while tile kt is consumed
  constexpr int TILE = FK * HeadDim<DH>::DHL;
  __shared__ __attribute__((aligned(1024))) bf16_t Kbuf[2 * TILE];
  __shared__ __attribute__((aligned(1024))) bf16_t Vbuf[2 * TILE];
  int seq, qt, nqt, tile_id, hq;
  tile_and_head(Hq, &tile_id, &hq, blockIdx.x);
  if (!find_tile(cu, ord, S, FQ, tile_id, &seq, &qt, &nqt)) return;
  const int hk = hq / group;
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  // keys and values may be packed on their own (a chunk of a context-parallel partition)
  const int lok = cuk[seq], Lk = cuk[seq + 1] - lok;
  const int q0 = qt * FQ;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int half = lane >> 5;
  const int qpos = q0 + wave * 32 + (lane & 31);          // this lane's query (column of S^T)
  const int qrow = min(qpos, L - 1);
  if (Lk == 0) {
    // no key in this chunk (workgroup-uniform): zero output, lse = -inf
    if (qpos < L) {
      bf16_t* op = o + (size_t)(lo + qpos) * ldo + hq * DH;
      for (int c = half * (DH / 2); c < (half + 1) * (DH / 2); c += 4) {
        bf16x4 z = {(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
        *reinterpret_cast<bf16x4*>(op + c) = z;
      }
      if (half == 0) lse[(size_t)hq * Ttot + lo + qpos] = -INFINITY;
    }
    return;
  }

  bf16x8 qf[HeadDim<DH>::KS];
  {
    const bf16_t* qp = q + (size_t)(lo + qrow) * ld + hq * DH;
#pragma unroll
    for (int ks = 0; ks < HeadDim<DH>::KS; ++ks) qf[ks] = load_chunk<DH>(qp, ks * 2 + half);
  }
  f32x16 oacc[HeadDim<DH>::NB];
#pragma unroll
  for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[j][r] = 0.f;
  float m = -INFINITY, lsum = 0.f;

  const int kend = CAUSAL ? min(Lk, q0 + FQ) : Lk;
  const int nkt = (kend + FK - 1) / FK;
  const bf16_t* kbase = k + (size_t)lok * ldk + hk * DH;
  const bf16_t* vbase = v + (size_t)lok * ldk + hk * DH;
  using Tile = TileAsync<FK, DH, 256>;
  Tile tile;
  tile.init(ldk, tid);
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    Tile::zero_padding(Kbuf + b * TILE, tid);
    Tile::zero_padding(Vbuf + b * TILE, tid);
  }
  tile.issue(kbase, ldk, Lk, Kbuf, wave_u);
  tile.issue(vbase, ldk, Lk, Vbuf, wave_u);
  settle_compiler_loads();                 // the Q fragments (and, with them, tile 0)

  // The step comes in two copies, without and with the per-element mask test, each in a loop of
  // its own: the leading key tiles lie wholly inside the sequence (and before the diagonal under a
  // causal mask) and need no test; written as a run-time condition inside the unrolled code, the
  // test becomes compare/select pairs that every step pays for.  Every wavefront runs nkt steps
  // in total (the split may differ between wavefronts; the barrier count per step does not).
  auto step = [&](int kt, auto masked, auto parity) {
    constexpr bool MASKED = decltype(masked)::value;
    constexpr int PAR = decltype(parity)::value;
    const bf16_t* Ks = Kbuf + PAR * TILE;
    const bf16_t* Vs = Vbuf + PAR * TILE;
    // one barrier per step: tile kt has landed for every wavefront, and every wavefront is done
    // with tile kt-1, whose buffer the loads of tile kt+1 overwrite
    wait_async_tiles();
    __syncthreads();
    if (kt + 1 < nkt) {
      const size_t next = (size_t)(kt + 1) * FK * ldk;
      tile.issue(kbase + next, ldk, Lk - (kt + 1) * FK, Kbuf + (1 - PAR) * TILE, wave_u);
      tile.issue(vbase + next, ldk, Lk - (kt + 1) * FK, Vbuf + (1 - PAR) * TILE, wave_u);
    }
    const int key0 = kt * FK;
    // S^T = K Q^T for both 32-key blocks first: the MFMAs of block 1 run while the
    // softmax arithmetic of block 0 occupies the vector unit, and the P V MFMAs of
    // block 0 run under the softmax of block 1.
    f32x16 sacc[FK / 32];
#pragma unroll
    for (int b = 0; b < FK / 32; ++b) sacc[b] = f32x16{};
    {
      // K fragments are requested from LDS AHEAD MFMAs before their use (a ring of register sets)
      constexpr int KS = HeadDim<DH>::KS, NSTEP = (FK / 32) * KS, AHEAD = 2;
      bf16x8 fk[AHEAD + 1];
#pragma unroll
      for (int n = 0; n < AHEAD && n < NSTEP; ++n) fk[n] = frag_rows<HeadDim<DH>::DHL>(Ks, (n / KS) * 32, n % KS, lane);
#pragma unroll
      for (int n = 0; n < NSTEP; ++n) {
        const int m = n + AHEAD;
        if (m < NSTEP) fk[m % (AHEAD + 1)] = frag_rows<HeadDim<DH>::DHL>(Ks, (m / KS) * 32, m % KS, lane);
        sacc[n / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[n % (AHEAD + 1)], qf[n % KS], sacc[n / KS], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // mask: keys past the sequence end, and keys after the query under a causal mask
#pragma unroll
    for (int b = 0; b < FK / 32; ++b) {
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (MASKED) {
          const int key = key0 + b * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
          if (key >= Lk || (CAUSAL && key > qpos)) sacc[b][r] = -INFINITY;
        }
        mx = fmaxf(mx, sacc[b][r]);
      }
      mx = max_with_other_half(mx) * scale_log2;
      // Lazy rescaling: the running maximum only moves (and O, l are only rescaled)
      // when some row's maximum grew by more than 2^8; until then probabilities are
      // taken relative to the older maximum (they stay below 2^8, exact in fp32).
      if (__builtin_amdgcn_ballot_w64(mx > m + 8.0f) != 0) {
        const float m_new = fmaxf(m, mx);
        const float corr = __builtin_amdgcn_exp2f(m - m_new);   // m = -inf at the start: 0
        m = m_new;
        lsum *= corr;
#pragma unroll
        for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[j][r] *= corr;
      }
      float psum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[b][r], scale_log2, -m));   // masked: exp2(-inf) = 0
        sacc[b][r] = p;
        psum += p;
      }
      lsum += psum;
      const bf16x8 p0 = acc_to_operand(sacc[b], 0), p1 = acc_to_operand(sacc[b], 1);
      // O^T += V^T P^T, the transposed V operands requested one pair of MFMAs ahead
      {
        constexpr int NB = HeadDim<DH>::NB;
        bf16x8 fr[2][2];
        fr[0][0] = frag_cols<HeadDim<DH>::DHL>(Vs, 0, b * 32, lane);
        fr[0][1] = frag_cols<HeadDim<DH>::DHL>(Vs, 0, b * 32 + 16, lane);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          if (j + 1 < NB) {
            fr[(j + 1) & 1][0] = frag_cols<HeadDim<DH>::DHL>(Vs, (j + 1) * 32, b * 32, lane);
            fr[(j + 1) & 1][1] = frag_cols<HeadDim<DH>::DHL>(Vs, (j + 1) * 32, b * 32 + 16, lane);
          }
          oacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][0], p0, oacc[j], 0, 0, 0);
          oacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][1], p1, oacc[j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // tiles kt < n_plain need no test: key0 + FK <= Lk, and key0 + FK - 1 <= this wavefront's first query
  int n_plain = Lk / FK;
  if (CAUSAL) n_plain = min(n_plain, (q0 + wave * 32 + 1) / FK);
  n_plain = min(n_plain, nkt);
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  for (int kt = 0; kt < nkt; ++kt) {
    const bool plain = kt < n_plain;
    if (kt & 1) { if (plain) step(kt, std::false_type{}, P1{}); else step(kt, std::true_type{}, P1{}); }
    else { if (plain) step(kt, std::false_type{}, P0{}); else step(kt, std::true_type{}, P0{}); }
  }
  lsum = sum_with_other_half(lsum);
  if (qpos < L) {
    const float inv = 1.0f / lsum;
    bf16_t* op = o + (size_t)(lo + qpos) * ldo + hq * DH;
#pragma unroll
    for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16_t)(oacc[j][g * 4 + e] * inv);
        if (DH % 32 == 0 || j * 32 + g * 8 + half * 4 < DH)
          *reinterpret_cast<bf16x4*>(op + j * 32 + g * 8 + half * 4) = w;
      }
    if (half == 0) lse[(size_t)hq * Ttot + lo + qpos] = (m + log2f(lsum)) * LN2;
  }
}

// ---- tiles whose reads are one lane constant plus an immediate offset (head sizes 64 and 128) ----------
// A run of 512 / DH rows is the 1 KiB that one load instruction of a wavefront fills.  In a run, 64-byte groups of
// four chunks lie row after row, and the runs are PAD bytes apart from each other, so that row reads and transpose
// reads are free of bank conflicts; for 64, the lowest bit of the chunk is turned in every second four rows.
template <int DH>
struct RunTile {
  static constexpr int RPR = 512 / DH, RUN = 1024 + (DH == 128 ? 16 : 32);
  static constexpr int bytes(int rows) { return rows / RPR * RUN; }
  // this lane's row (in the run) and 16-byte chunk in a load
  static __device__ inline int load_row(int l) { return (l >> 2) & (RPR - 1); }
  static __device__ inline int load_chunk(int l) {
    return DH == 128 ? (l >> 4) * 4 + (l & 3) : (l >> 5) * 4 + ((l & 3) ^ ((l >> 4) & 1));
  }
  // operand with rows as MFMA rows: lane l holds row l % 32 of a block, dh = ks * 16 + (l / 32) * 8 .. + 7
  static __device__ inline int rows_at(int l) {
    const int r = l & 31, half = l >> 5;
    return r / RPR * RUN + (r & (RPR - 1)) * 64 + (DH == 128 ? half : half ^ ((r >> 2) & 1)) * 16;
  }
  static constexpr int rows_imm(int block, int ks) { return block * (32 / RPR) * RUN + (ks >> 1) * (RPR * 64) + (ks & 1) * 32; }
  // transposed operand: MFMA row = dh index j * 32 + l % 32, k index = tile rows r16 * 16 .. (see frag_cols)
  static __device__ inline int cols_at(int l) {
    const int gi = l >> 4, s = l & 15, c = (gi & 1) * 2 + ((s & 3) >> 1);
    return DH == 128 ? (gi >> 1) * RUN + (s >> 2) * 64 + c * 16 + (s & 1) * 8
                     : ((gi >> 1) * 4 + (s >> 2)) * 64 + (c ^ (gi >> 1)) * 16 + (s & 1) * 8;
  }
  static constexpr int cols_imm(int j, int r16) { return j * (RPR * 64) + r16 * (16 / RPR) * RUN; }
  static __device__ inline bf16x8 read_rows(const unsigned char* base, int block, int ks) {
    return *reinterpret_cast<const bf16x8*>(base + rows_imm(block, ks));
  }
  static __device__ inline bf16x8 read_cols(const unsigned char* base, int j, int r16) {
    const unsigned char* a = base + cols_imm(j, r16);
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)a);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(a + 8 / RPR * RUN));
    union { struct { s16x4 a, b; } s; bf16x8 v; } u;
    u.s.a = lo; u.s.b = hi;
    return u.v;
  }
};

__device__ inline const bf16_t* scalar_ptr(const void* p) {
  const uint64_t b = reinterpret_cast<uint64_t>(p);
  return reinterpret_cast<const bf16_t*>(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32) |
                                         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b));
}

// end of a phase: this wavefront's LDS accesses are done, then the workgroup meets
__device__ inline void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Forward with two groups of wavefronts that take turns (head sizes 64 and 128, long sequences): wavefronts w and
// w + 4 share a SIMD, and while one multiplies -- P V of a key tile, then Q K of the next -- the other one does
// the softmax of its tile.  Left to themselves (two workgroups of four wavefronts), two wavefronts of a SIMD
// often want the same unit: matrix pipe busy 50 % of the cycles at head size 128, vector unit 56 %.
// Two workgroups of four wavefronts -> this, us: 4 x 4096 bidirectional, 16 heads of 128, 577 -> 482 (1140 TFLOP/s), of
// 64, 369 -> 330; 32768 tokens of causal documents, 32 / 8 heads of 128, 2914 -> 2501; 16 samples of about 1130, 24 heads,
// 360 -> 327.  Bound by the vector unit at head size 64 (78 % busy before) and by power at 128.
constexpr int AQ = 256;   // query rows per workgroup

template <int DH, bool CAUSAL>
__global__ __launch_bounds__(512, 2) void fa_fwd_alt_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk, int S,
    bf16_t* __restrict__ o, int ldo, float* __restrict__ lse, int Ttot, int Hq, int group,
    float scale_log2, SeqOrder ord) {
  using RT = RunTile<DH>;
  constexpr int KS = DH / 16, NB = DH / 32, KBL = FK / 32, TILE = RT::bytes(FK), RUNS = FK / RT::RPR / 8;
  constexpr int RING = 3;
  __shared__ __attribute__((aligned(1024))) unsigned char Kbuf[RING * TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char Vbuf[RING * TILE];
  int seq, qt, nqt, tile_id, hq;
  tile_and_head(Hq, &tile_id, &hq, blockIdx.x);
  if (!find_tile(cu, ord, S, AQ, tile_id, &seq, &qt, &nqt)) return;
  const int hk = hq / group;
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  const int lok = cuk[seq], Lk = cuk[seq + 1] - lok;
  const int q0 = qt * AQ;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qfirst = q0 + wave * 32;
  const int qpos = qfirst + (lane & 31);                  // this lane's query (column of S^T)
  bf16x8 qf[KS];
  {
    const bf16_t* qp = q + (size_t)(lo + min(qpos, L - 1)) * ld + hq * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[ks] = load_chunk<DH>(qp, ks * 2 + half);
  }
  f32x16 oacc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) oacc[j] = f32x16{};
  float m = -INFINITY, lsum = 0.f;
  // key tiles of the workgroup, and those of this wavefront (none if its queries lie past the sequence)
  const int nkt = ((CAUSAL ? min(Lk, q0 + AQ) : Lk) + FK - 1) / FK;
  const int mine = qfirst >= L ? 0 : CAUSAL ? min(nkt, (qfirst + 31) / FK + 1) : nkt;
  const int plain = CAUSAL ? min(Lk / FK, (qfirst + 1) / FK) : Lk / FK;   // leading tiles that need no mask test
  const bf16_t* kbase = scalar_ptr(k + (size_t)lok * ldk + hk * DH);
  const bf16_t* vbase = scalar_ptr(v + (size_t)lok * ldk + hk * DH);
  const uint32_t klds = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)Kbuf;
  const uint32_t vlds = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)Vbuf;
  const uint32_t lrow = RT::load_row(lane), lchunk = RT::load_chunk(lane) * 16;
  // tile t of K or V into ring slot `slot` (t % 3); rows past the keys are clamped (their P is 0)
  auto fetch = [&](const bf16_t* base, uint32_t lds, int t, int slot) {
    if (t >= nkt) return;
    const bf16_t* src = base + (size_t)t * FK * ldk;
    const int last = Lk - t * FK - 1;
    const uint32_t dst = lds + slot * TILE;
#pragma unroll
    for (int i = 0; i < RUNS; ++i) {
      const int r = wave * RUNS + i;
      const uint32_t off = (uint32_t)min(r * RT::RPR + (int)lrow, last) * (uint32_t)ldk * 2u + lchunk;
      TileAsync<FK, DH, 512>::load16(src, off, dst + r * RT::RUN);
    }
  };
  f32x16 sacc[KBL];
  bf16x8 pb[KBL][2];
  static_assert(KBL == 2, "one factor between the blocks of a tile");
  bool late = false;                                      // the maximum moved in the tile's second block, by late_corr
  float late_corr = 1.f;
  const int rows_at = RT::rows_at(lane), cols_at = RT::cols_at(lane);
  auto scores = [&](int slot) {                           // S^T = K Q^T of the key tile in a ring slot
    int at = slot * TILE + rows_at;
    asm volatile("" : "+v"(at));                           // one register; the rest is immediates
    const unsigned char* base = Kbuf + at;
    constexpr int NSTEP = KBL * KS, AHEAD = 3;
    bf16x8 f[AHEAD + 1];
#pragma unroll
    for (int b = 0; b < KBL; ++b) sacc[b] = f32x16{};
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) f[n] = RT::read_rows(base, n % KBL, n / KBL);
#pragma unroll
    for (int n = 0; n < NSTEP; ++n) {
      if (n + AHEAD < NSTEP) f[(n + AHEAD) % (AHEAD + 1)] = RT::read_rows(base, (n + AHEAD) % KBL, (n + AHEAD) / KBL);
      sacc[n % KBL] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[n % (AHEAD + 1)], qf[n / KBL], sacc[n % KBL], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto values = [&](int slot) {                           // O^T += V^T P^T
    int at = slot * TILE + cols_at;
    asm volatile("" : "+v"(at));
    const unsigned char* base = Vbuf + at;
    constexpr int NSTEP = KBL * 2 * NB, AHEAD = 3;         // step n: 16 keys n / NB, 32 columns n % NB
    bf16x8 f[AHEAD + 1];
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) f[n] = RT::read_cols(base, n % NB, n / NB);
#pragma unroll
    for (int n = 0; n < NSTEP; ++n) {
      if (n == 2 * NB && late) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) oacc[j][r] *= late_corr;
      }
      if (n + AHEAD < NSTEP) f[(n + AHEAD) % (AHEAD + 1)] = RT::read_cols(base, (n + AHEAD) % NB, (n + AHEAD) / NB);
      oacc[n % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[n % (AHEAD + 1)], pb[n / NB / 2][n / NB % 2], oacc[n % NB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto softmax = [&](int t) {
    if (t >= plain) {
      asm volatile("");                                    // keeps the tests out of the tiles that need none
      // element (b, r): key t * 64 + b * 32 + (r / 4) * 8 + half * 4 + r % 4
      const int left = Lk - t * FK - half * 4, ahead = qpos - t * FK - half * 4;
#pragma unroll
      for (int b = 0; b < KBL; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int e = b * 32 + (r >> 2) * 8 + (r & 3);
          if (e >= left || (CAUSAL && e > ahead)) sacc[b][r] = -INFINITY;
        }
    }
    late = false;
#pragma unroll
    for (int b = 0; b < KBL; ++b) {
      float mx = -INFINITY;
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sacc[b][r]);
      mx = max_with_other_half(mx) * scale_log2;
      // lazy rescaling, as in the kernel above; the output takes the factor of a later block between the
      // blocks' products (see values)
      if (__builtin_amdgcn_ballot_w64(mx > m + 8.0f) != 0) {
        const float m_new = fmaxf(m, mx);
        const float corr = __builtin_amdgcn_exp2f(m - m_new);   // m = -inf at the start: 0
        m = m_new;
        lsum *= corr;
        if (b == 0) {
#pragma unroll
          for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[j][r] *= corr;
        } else {
          late = true;
          late_corr = corr;
        }
      }
      float psum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[b][r], scale_log2, -m));   // masked: exp2(-inf) = 0
        sacc[b][r] = p;
        psum += p;
      }
      lsum += psum;
      pb[b][0] = acc_to_operand(sacc[b], 0);
      pb[b][1] = acc_to_operand(sacc[b], 1);
    }
  };
  settle_compiler_loads();                                // Q fragments, offsets
  fetch(kbase, klds, 0, 0);
  fetch(vbase, vlds, 0, 0);
  fetch(kbase, klds, 1, 1);
  wait_async_tiles();
  phase_barrier();
  if (wave >= 4) phase_barrier();                         // the second group stays one phase behind
  if (mine > 0) scores(0);
  phase_barrier();
  for (int t = 0, s0 = 0, s1 = 1, s2 = 2; t < nkt; ++t) {   // ring slots of tiles t, t + 1, t + 2
    // both groups are past the tiles these overwrite (V t - 2, K t - 1); they are read two phases from now
    fetch(vbase, vlds, t + 1, s1);
    fetch(kbase, klds, t + 2, s2);
    if (t < mine) softmax(t);
    phase_barrier();
    if (t < mine) values(s0);
    if (t + 1 < mine) scores(s1);
    wait_async_tiles();
    phase_barrier();
    const int s = s0;
    s0 = s1; s1 = s2; s2 = s;
  }
  if (wave < 4) phase_barrier();
  lsum = sum_with_other_half(lsum);
  if (qpos < L) {
    // no key in this chunk: zero output, lse = -inf
    const float inv = Lk > 0 ? 1.0f / lsum : 0.f;
    bf16_t* op = o + (size_t)(lo + qpos) * ldo + hq * DH;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16_t)(oacc[j][g * 4 + e] * inv);
        *reinterpret_cast<bf16x4*>(op + j * 32 + g * 8 + half * 4) = w;
      }
    if (half == 0) lse[(size_t)hq * Ttot + lo + qpos] = Lk > 0 ? (m + log2f(lsum)) * LN2 : -INFINITY;
  }
}

int count_tiles(const int32_t* cu_host, int S, int rows) {
  long n = 0;
  for (int s = 0; s < S; ++s) n += (cu_host[s + 1] - cu_host[s] + rows - 1) / rows;
  return (int)n;
}

// keys a query walks on average
double keys_per_query(const AttnArgs& a) {
  const int32_t* ck = a.kv_cu_host();
  double pairs = 0;
  for (int s = 0; s < a.S; ++s) pairs += (double)(a.cu_host[s + 1] - a.cu_host[s]) * (ck[s + 1] - ck[s]);
  return a.T > 0 ? (a.causal ? 0.5 : 1.0) * pairs / a.T : 0.0;
}

// 256-row tiles and alternating groups, or 128-row tiles and two workgroups per CU?  The former where they cut the
// sequences about as well and come to two per CU or more, and
//  - where a query walks enough keys to pay for the turns' start and end.  Forward, 128 -> 256 rows, us: head size 128,
//    bidirectional, 24 x 256, 32 heads, 55 -> 62; 16 x 512, 24 heads, 74 -> 78; 4 x 2048, 24 heads, 217 -> 197; causal 12 x 520,
//    24 heads, 60 -> 70; 8 documents of 411 to 1800, 32 heads, 128 -> 122.  Head size 64, bidirectional, 4 x 900, 32 heads, 48 -> 44.
//  - under a full mask, where the last round is nearly full, since all tiles of a sequence take equally long: head size 64,
//    8 x 768, 24 heads (2.25 rounds), 47 -> 52; 128, 6 x 1000, 16 heads (1.5 rounds), 65 -> 69.
//  - not at head size 64 under a causal mask, where the vector unit bounds both and long tiles cannot be evened out: 4 x 2048,
//    16 heads, 66 -> 72; 2 x 2600, 24 heads, 73 -> 87; ahead only with 64 heads (4096, 172 -> 157).
// 189 packs of 577 to 18432 tokens, both masks, 16 to 64 heads: no choice of 256 rows is more than 4 % behind 128.
bool queries_alternating(const AttnArgs& a) {
  if (a.causal && a.dh == 64) return false;
  const long ta = count_tiles(a.cu_host, a.S, AQ), tn = count_tiles(a.cu_host, a.S, FQ), wgs = ta * a.Hq;
  if (wgs < 2 * NUM_CU || ta * 8 > tn * 5) return false;
  if (a.causal) return keys_per_query(a) >= 600;
  return keys_per_query(a) >= 800 && (long)cdiv(wgs, NUM_CU) * NUM_CU * 4 <= wgs * 5;
}

template <int DH>
bm_status fwd_launch(const AttnArgs& a, void* o, float* lse, hipStream_t st) {
  const float sl2 = LOG2E / sqrtf((float)a.dh);
  if constexpr (DH != 72) {
    if (queries_alternating(a)) {
      const dim3 grid(count_tiles(a.cu_host, a.S, AQ) * a.Hq);
      const SeqOrder ord = make_seq_order(a.cu_host, a.kv_cu_host(), a.S, AQ, !a.causal);
      auto kern = fa_fwd_alt_kernel<DH, false>;
      if constexpr (DH == 128) if (a.causal) kern = fa_fwd_alt_kernel<DH, true>;
      hipLaunchKernelGGL(kern, grid, dim3(512), 0, st, (const bf16_t*)a.q, (const bf16_t*)a.k, (const bf16_t*)a.v,
                         a.ld_qkv, a.kv_ld(), a.cu_dev, a.kv_cu_dev(), a.S, (bf16_t*)o, a.Hq * a.dh, lse, a.T, a.Hq,
                         a.Hq / a.Hkv, sl2, ord);
      BM_CHECK_LAUNCH("fa_fwd_alt");
      return BM_OK;
    }
  }
  dim3 grid(count_tiles(a.cu_host, a.S, FQ) * a.Hq), block(256);
  if (grid.x == 0) return BM_OK;
  // a query tile runs as long as its sequence has keys
  const SeqOrder ord = make_seq_order(a.cu_host, a.kv_cu_host(), a.S, FQ, !a.causal);
#define BM_L(C)                                                                                  \
  hipLaunchKernelGGL((fa_fwd_kernel<DH, C>), grid, block, 0, st, (const bf16_t*)a.q,             \
                     (const bf16_t*)a.k, (const bf16_t*)a.v, a.ld_qkv, a.kv_ld(), a.cu_dev,      \
                     a.kv_cu_dev(), a.S, (bf16_t*)o, a.Hq * a.dh, lse, a.T, a.Hq, a.Hq / a.Hkv, sl2, ord)
  if (a.causal) BM_L(true); else BM_L(false);
#undef BM_L
  BM_CHECK_LAUNCH("fa_fwd");
  return BM_OK;
}

// =============================================================================
// backward
// =============================================================================
// delta[h, t] = sum_c dO[t,h,c] * O[t,h,c]; 8 (head size 64) or 16 lanes share one (row, head),
// 16 bytes each, so a wavefront reads whole contiguous row segments
template <int DH> struct DeltaLanes { static constexpr int N = DH <= 64 ? 8 : 16, SHIFT = DH <= 64 ? 3 : 4; };
template <int DH>
__global__ void fa_delta_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o, int ldo,
                                float* __restrict__ delta, int Ttot, int Hq) {
  constexpr int LP = DeltaLanes<DH>::N;
  const long gid = ((long)blockIdx.x * blockDim.x + threadIdx.x) >> DeltaLanes<DH>::SHIFT;
  const int c = (threadIdx.x & (LP - 1)) * 8;
  float s = 0.f;
  const bool live = gid < (long)Ttot * Hq;
  const int t = live ? (int)(gid / Hq) : 0, hq = live ? (int)(gid % Hq) : 0;
  if (live && c < DH) {
    float a[8], b[8];
    load16(o + (size_t)t * ldo + hq * DH + c, a);
    load16(d_o + (size_t)t * ldo + hq * DH + c, b);
#pragma unroll
    for (int e = 0; e < 8; ++e) s = fmaf(a[e], b[e], s);
  }
#pragma unroll
  for (int off = LP / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  if (live && c == 0) delta[(size_t)hq * Ttot + t] = s;
}

constexpr int WIDE_KEYS = 256;  // keys per workgroup of the wide dK/dV kernel
constexpr int BK_KEYS = 128;   // keys per workgroup in the dK/dV kernel (32 per wavefront)
constexpr int BK_Q = 64;       // query rows per step

// dK, dV of one 128-key tile of one kv head: walks the q heads of the group and the
// query tiles; scores are kept as S[q, key] so that P and dS are B operands as they are.
template <int DH> constexpr int dkdv_lds_bytes() { return 4 * BK_Q * HeadDim<DH>::DHL * 2 + 4 * BK_Q * 4; }
template <int DH, bool CAUSAL>
__device__ inline void dkdv_tile(unsigned char* lds, int block, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cuq, const int32_t* __restrict__ cu,
    int S, bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int ldd, int Tq, int Ttot, int Hkv, int group,
    float scale, float scale_log2, int gsplit,
    float* __restrict__ part /* [gsplit][2][Ttot][Hkv*DH] fp32 when gsplit > 1 */, SeqOrder ord) {
  // cu, Ttot, ldk: the packing of the keys/values (and of dk, dv); cuq, Tq, ld: of the queries
  // Q and dO tiles are double-buffered and streamed into LDS (see TileAsync)
  constexpr int TILE = BK_Q * HeadDim<DH>::DHL;
  bf16_t* const Qbuf = reinterpret_cast<bf16_t*>(lds);
  bf16_t* const Dbuf = Qbuf + 2 * TILE;
  float* const Lbuf = reinterpret_cast<float*>(Dbuf + 2 * TILE);
  float* const Dlbuf = Lbuf + 2 * BK_Q;
  int seq, kt, nkt, tile_id, hk;
  // with gsplit > 1 a workgroup takes group/gsplit of the q heads that share this kv head
  // and leaves an fp32 partial; the (kv head, q-head part) pair plays the head's role
  int hk_gs;
  tile_and_head(Hkv * gsplit, &tile_id, &hk_gs, block);
  hk = hk_gs / gsplit;
  const int gs = hk_gs % gsplit;
  const int gpart = group / gsplit;
  if (!find_tile(cu, ord, S, BK_KEYS, tile_id, &seq, &kt, &nkt)) return;
  kt = nkt - 1 - kt;                                   // early key tiles see the most queries
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  const int loq = cuq[seq], Lq = cuq[seq + 1] - loq;
  const int kb0 = kt * BK_KEYS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int kpos = kb0 + wave * 32 + (lane & 31);       // this lane's key (column of S)
  const int krow = min(kpos, L - 1);

  // With several resident wavefronts to hide the LDS read, dP starts at -delta of its query row, so that the
  // MFMAs leave dP - delta.  (With one wavefront per SIMD the read in front of the MFMAs costs more.)
  constexpr bool FOLD_DELTA = DH <= 64;
  bf16x8 kf[HeadDim<DH>::KS], vf[HeadDim<DH>::KS];
  {
    const bf16_t* kp = k + (size_t)(lo + krow) * ldk + hk * DH;
    const bf16_t* vp = v + (size_t)(lo + krow) * ldk + hk * DH;
#pragma unroll
    for (int ks = 0; ks < HeadDim<DH>::KS; ++ks) {
      kf[ks] = load_chunk<DH>(kp, ks * 2 + half);
      vf[ks] = load_chunk<DH>(vp, ks * 2 + half);
    }
  }
  f32x16 dkacc[HeadDim<DH>::NB], dvacc[HeadDim<DH>::NB];
#pragma unroll
  for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dkacc[j][r] = 0.f; dvacc[j][r] = 0.f; }

  const int qstart = CAUSAL ? (kb0 / BK_Q) * BK_Q : 0;
  const int nqt = Lq > qstart ? (Lq - qstart + BK_Q - 1) / BK_Q : 0;   // no query: dk = dv = 0
  const int iters = nqt * gpart;
  using Tile = TileAsync<BK_Q, DH, 256>;
  Tile tq, td;
  tq.init(ld, tid);
  td.init(ldo, tid);
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  float st_l = 0.f, st_d = 0.f;
  auto fetch = [&](int it, int par) {
    const int hq = hk * group + gs * gpart + it / nqt;
    const int q0 = qstart + (it % nqt) * BK_Q;
    tq.issue(q + ((size_t)loq + q0) * ld + hq * DH, ld, Lq - q0, Qbuf + par * TILE, wave_u);
    td.issue(d_o + ((size_t)loq + q0) * ldo + hq * DH, ldo, Lq - q0, Dbuf + par * TILE, wave_u);
    if (tid < BK_Q) {
      const int qi = min(q0 + tid, Lq - 1);
      st_l = lse[(size_t)hq * Tq + loq + qi];      // used (and waited for) when the next step opens
      st_d = delta[(size_t)hq * Tq + loq + qi];
    }
  };
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    Tile::zero_padding(Qbuf + b * TILE, tid);
    Tile::zero_padding(Dbuf + b * TILE, tid);
  }
  if (iters > 0) fetch(0, 0);
  settle_compiler_loads();                              // K and V fragments, lse, delta (and, with them, tile 0)
  // one step; MASKED is a compile-time copy with the per-element tests (see the forward kernel)
  auto step = [&](int it, auto masked, auto parity) {
    constexpr bool MASKED = decltype(masked)::value;
    constexpr int PAR = decltype(parity)::value;
    const bf16_t* Qs = Qbuf + PAR * TILE;
    const bf16_t* Ds = Dbuf + PAR * TILE;
    const float* Ls = Lbuf + PAR * BK_Q;
    const float* Dl = Dlbuf + PAR * BK_Q;
    if (tid < BK_Q) { Lbuf[PAR * BK_Q + tid] = st_l * LOG2E; Dlbuf[PAR * BK_Q + tid] = st_d; }
    wait_async_tiles();
    __syncthreads();      // tile `it` is there for everyone, and everyone is done with tile it-1
    if (it + 1 < iters) fetch(it + 1, 1 - PAR);
    const int q0 = qstart + (it % nqt) * BK_Q;
    // S = Q K^T and dP = dO V^T for both 32-query blocks first, then per block the
    // softmax arithmetic (under the other block's MFMAs) followed by its dV / dK MFMAs.
    f32x16 sacc[BK_Q / 32], dpacc[BK_Q / 32];
#pragma unroll
    for (int qb = 0; qb < BK_Q / 32; ++qb) {
      sacc[qb] = f32x16{};
      if (!FOLD_DELTA) dpacc[qb] = f32x16{};
      if (FOLD_DELTA) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(Dl + qb * 32 + g * 8 + half * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) dpacc[qb][g * 4 + e] = -d4[e];
        }
      }
    }
    {
      // the operand fragments of step n + AHEAD are requested from LDS before the MFMAs of step n
      // are issued (a ring of AHEAD + 1 register sets): with one wavefront per SIMD nothing else
      // would cover the LDS latency in front of every MFMA
      constexpr int KS = HeadDim<DH>::KS, NSTEP = (BK_Q / 32) * KS, AHEAD = 2;
      bf16x8 fq[AHEAD + 1], fd[AHEAD + 1];
#pragma unroll
      for (int n = 0; n < AHEAD && n < NSTEP; ++n) {
        fq[n] = frag_rows<HeadDim<DH>::DHL>(Qs, (n / KS) * 32, n % KS, lane);
        fd[n] = frag_rows<HeadDim<DH>::DHL>(Ds, (n / KS) * 32, n % KS, lane);
      }
#pragma unroll
      for (int n = 0; n < NSTEP; ++n) {
        const int qb = n / KS, ks = n % KS, m = n + AHEAD;
        if (m < NSTEP) {
          fq[m % (AHEAD + 1)] = frag_rows<HeadDim<DH>::DHL>(Qs, (m / KS) * 32, m % KS, lane);
          fd[m % (AHEAD + 1)] = frag_rows<HeadDim<DH>::DHL>(Ds, (m / KS) * 32, m % KS, lane);
        }
        sacc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fq[n % (AHEAD + 1)], kf[ks], sacc[qb], 0, 0, 0);
        dpacc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fd[n % (AHEAD + 1)], vf[ks], dpacc[qb], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int qb = 0; qb < BK_Q / 32; ++qb) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int qoff = qb * 32 + g * 8 + half * 4;
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(Ls + qoff);
        f32x4 d4 = {0.f, 0.f, 0.f, 0.f};
        if (!FOLD_DELTA) d4 = *reinterpret_cast<const f32x4*>(Dl + qoff);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int r = g * 4 + e;
          float p = __builtin_amdgcn_exp2f(fmaf(sacc[qb][r], scale_log2, -l4[e]));
          if (MASKED) {
            const int qi = q0 + qoff + e;
            if (qi >= Lq || kpos >= L || (CAUSAL && kpos > qi)) p = 0.f;
          }
          sacc[qb][r] = p;
          dpacc[qb][r] = FOLD_DELTA ? p * dpacc[qb][r] : p * (dpacc[qb][r] - d4[e]);
        }
      }
      const bf16x8 p0 = acc_to_operand(sacc[qb], 0), p1 = acc_to_operand(sacc[qb], 1);
      const bf16x8 s0 = acc_to_operand(dpacc[qb], 0), s1 = acc_to_operand(dpacc[qb], 1);
      {
        // dV += dO^T P, dK += Q^T dS: 4 MFMAs per 32 columns of dh, their transposed operands
        // requested one group ahead
        constexpr int NB = HeadDim<DH>::NB;
        bf16x8 fr[2][4];
        auto request = [&](int j, bf16x8 (&f)[4]) {
          f[0] = frag_cols<HeadDim<DH>::DHL>(Ds, j * 32, qb * 32, lane);
          f[1] = frag_cols<HeadDim<DH>::DHL>(Ds, j * 32, qb * 32 + 16, lane);
          f[2] = frag_cols<HeadDim<DH>::DHL>(Qs, j * 32, qb * 32, lane);
          f[3] = frag_cols<HeadDim<DH>::DHL>(Qs, j * 32, qb * 32 + 16, lane);
        };
        request(0, fr[0]);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          if (j + 1 < NB) request(j + 1, fr[(j + 1) & 1]);
          dvacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][0], p0, dvacc[j], 0, 0, 0);
          dvacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][1], p1, dvacc[j], 0, 0, 0);
          dkacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][2], s0, dkacc[j], 0, 0, 0);
          dkacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][3], s1, dkacc[j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // Which query tiles need the tests: all of them when this key tile is cut by the sequence end;
  // else, per q head, the first ones under a causal mask (queries before this wavefront's last
  // key) and the last one when it is cut by the sequence end.  Every wavefront runs `iters`
  // steps; only the split between the copies differs.
  {
    // (one call site per copy of the step: with two the compiler stops inlining them)
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    const bool all_masked = kb0 + BK_KEYS > L;
    const int n_front = CAUSAL ? min(nqt, (wave * 32 + 32 + BK_Q - 1) / BK_Q) : 0;
    const int n_whole = max(n_front, (Lq - qstart) % BK_Q ? nqt - 1 : nqt);
    for (int it = 0, t = 0; it < iters; ++it, t = (t + 1 == nqt ? 0 : t + 1)) {
      const bool masked = all_masked || t < n_front || t >= n_whole;
      if (it & 1) { if (masked) step(it, std::true_type{}, P1{}); else step(it, std::false_type{}, P1{}); }
      else { if (masked) step(it, std::true_type{}, P0{}); else step(it, std::false_type{}, P0{}); }
    }
  }
  if (kpos < L && gsplit > 1) {
    const size_t plane = (size_t)Ttot * Hkv * DH;
    float* pk = part + ((size_t)gs * 2 + 0) * plane + (size_t)(lo + kpos) * (Hkv * DH) + hk * DH;
    float* pv = part + ((size_t)gs * 2 + 1) * plane + (size_t)(lo + kpos) * (Hkv * DH) + hk * DH;
#pragma unroll
    for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (DH % 32 == 0 || j * 32 + g * 8 + half * 4 < DH) {
          *reinterpret_cast<f32x4*>(pk + j * 32 + g * 8 + half * 4) =
              f32x4{dkacc[j][g * 4] * scale, dkacc[j][g * 4 + 1] * scale, dkacc[j][g * 4 + 2] * scale, dkacc[j][g * 4 + 3] * scale};
          *reinterpret_cast<f32x4*>(pv + j * 32 + g * 8 + half * 4) =
              f32x4{dvacc[j][g * 4], dvacc[j][g * 4 + 1], dvacc[j][g * 4 + 2], dvacc[j][g * 4 + 3]};
        }
  } else if (kpos < L) {
    bf16_t* pk = dk + (size_t)(lo + kpos) * ldd + hk * DH;
    bf16_t* pv = dv + (size_t)(lo + kpos) * ldd + hk * DH;
#pragma unroll
    for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 wk, wv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          wk[e] = (bf16_t)(dkacc[j][g * 4 + e] * scale);
          wv[e] = (bf16_t)dvacc[j][g * 4 + e];
        }
        if (DH % 32 == 0 || j * 32 + g * 8 + half * 4 < DH) {
          *reinterpret_cast<bf16x4*>(pk + j * 32 + g * 8 + half * 4) = wk;
          *reinterpret_cast<bf16x4*>(pv + j * 32 + g * 8 + half * 4) = wv;
        }
      }
  }
}

// dK, dV at head sizes above 64, where one wavefront cannot hold both accumulators next to a
// second resident wavefront: every 32-key block of the 128-key tile is shared by a PAIR of
// wavefronts that sit on the same SIMD (wavefronts w and w+4 of the 512-thread workgroup).
//   role 0 ("value" wavefront): S = Q K^T -> P = exp2(S*scale - lse), hands P to its partner
//                               through LDS, dV += dO^T P
//   role 1 ("key" wavefront):   dP = dO V^T, takes P, dS = P (dP - delta), dK += Q^T dS
// Each wavefront keeps one accumulator and one of K / V in registers (about 200 registers), so
// two are resident per SIMD and one's vector work runs under the other's MFMAs.  P travels as
// bf16 in the operand layout: role 0 feeds exactly these values to its own MFMAs, and role 1
// owns the same (key, query) elements in the same lanes, so the exchange is lane-private.
template <int DH> constexpr int dkdv_pair_lds_bytes() { return 4 * BK_Q * HeadDim<DH>::DHL * 2 + 4 * (BK_Q / 32) * 2 * 64 * 16 + 4 * BK_Q * 4; }
template <int DH, bool CAUSAL>
__device__ inline void dkdv_pair_tile(
    unsigned char* lds, int block, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cuq, const int32_t* __restrict__ cu,
    int S, bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int ldd, int Tq, int Ttot, int Hkv, int group,
    float scale, float scale_log2, int gsplit,
    float* __restrict__ part /* [gsplit][2][Ttot][Hkv*DH] fp32 when gsplit > 1 */, SeqOrder ord) {
  constexpr int DHL = HeadDim<DH>::DHL, KS = HeadDim<DH>::KS, NB = HeadDim<DH>::NB, NQB = BK_Q / 32;
  // Q and dO tiles are double-buffered and streamed into LDS (see TileAsync): with one workgroup
  // per CU nothing else runs while a tile is parked between two barriers
  constexpr int TILE = BK_Q * DHL;
  // (in this order: with lse and delta behind 64 KiB, out of an immediate offset's reach, the bidirectional kernel of
  // head size 128 spills 22 registers)
  bf16_t* const Qbuf = reinterpret_cast<bf16_t*>(lds);
  bf16_t* const Ps = Qbuf + 2 * TILE;                    // [key block][q block][half k-step][lane] x 16 B
  float* const Lbuf = reinterpret_cast<float*>(Ps + 4 * NQB * 2 * 64 * 8);
  float* const Dlbuf = Lbuf + 2 * BK_Q;
  bf16_t* const Dbuf = reinterpret_cast<bf16_t*>(Dlbuf + 2 * BK_Q);
  int seq, kt, nkt, tile_id, hk, hk_gs;
  tile_and_head(Hkv * gsplit, &tile_id, &hk_gs, block);
  hk = hk_gs / gsplit;
  const int gs = hk_gs % gsplit;
  const int gpart = group / gsplit;
  if (!find_tile(cu, ord, S, BK_KEYS, tile_id, &seq, &kt, &nkt)) return;
  kt = nkt - 1 - kt;                                   // early key tiles see the most queries
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  const int loq = cuq[seq], Lq = cuq[seq + 1] - loq;
  const int kb0 = kt * BK_KEYS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int kb = wave & 3, role = wave >> 2;            // wavefronts w and w+4 share a SIMD
  const int tid_r = tid & 255;                          // index inside the role's 256 threads
  const int kpos = kb0 + kb * 32 + (lane & 31);         // this lane's key (column of S)
  const int krow = min(kpos, L - 1);

  // role 0 keeps K (for S), role 1 keeps V (for dP)
  bf16x8 kvf[KS];
  {
    const bf16_t* p = (role == 0 ? k : v) + (size_t)(lo + krow) * ldk + hk * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kvf[ks] = load_chunk<DH>(p, ks * 2 + half);
  }
  f32x16 acc[NB];                                       // role 0: dV^T, role 1: dK^T (unscaled)
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;

  const int qstart = CAUSAL ? (kb0 / BK_Q) * BK_Q : 0;
  const int nqt = Lq > qstart ? (Lq - qstart + BK_Q - 1) / BK_Q : 0;   // no query: dk = dv = 0
  const int iters = nqt * gpart;
  // role 0's wavefronts bring in the Q tile, role 1's the dO tile; lse and delta of the tile's
  // queries pass through registers of the first wavefront
  using Tile = TileAsync<BK_Q, DH, 256>;
  Tile tile;
  tile.init(role == 0 ? ld : ldo, tid_r);
  const int wave_r = __builtin_amdgcn_readfirstlane(wave & 3);
  const int role_u = __builtin_amdgcn_readfirstlane(role);
  float st_l = 0.f, st_d = 0.f;
  auto fetch = [&](int it, int par) {
    const int hq = hk * group + gs * gpart + it / nqt;
    const int q0 = qstart + (it % nqt) * BK_Q;
    if (role_u == 0) tile.issue(q + ((size_t)loq + q0) * ld + hq * DH, ld, Lq - q0, Qbuf + par * TILE, wave_r);
    else tile.issue(d_o + ((size_t)loq + q0) * ldo + hq * DH, ldo, Lq - q0, Dbuf + par * TILE, wave_r);
    if (tid < BK_Q) {
      const int qi = min(q0 + tid, Lq - 1);
      st_l = lse[(size_t)hq * Tq + loq + qi];     // used (and waited for) when the next step opens
      st_d = delta[(size_t)hq * Tq + loq + qi];
    }
  };
#pragma unroll
  for (int b = 0; b < 2; ++b) Tile::zero_padding((role == 0 ? Qbuf : Dbuf) + b * TILE, tid_r);
  if (iters > 0) fetch(0, 0);
  settle_compiler_loads();                              // K / V fragments, lse, delta (and, with them, tile 0)
  bf16_t* my_p = Ps + (size_t)kb * (NQB * 2 * 64 * 8) + lane * 8;

  auto step = [&](int it, auto masked, auto parity) {
    constexpr bool MASKED = decltype(masked)::value;
    constexpr int PAR = decltype(parity)::value;
    const bf16_t* Qs = Qbuf + PAR * TILE;
    const bf16_t* Ds = Dbuf + PAR * TILE;
    const float* Ls = Lbuf + PAR * BK_Q;
    const float* Dl = Dlbuf + PAR * BK_Q;
    const bf16_t* rows_src = role == 0 ? Qs : Ds;       // phase 1 operand: Q (S) or dO (dP)
    const bf16_t* cols_src = role == 0 ? Ds : Qs;       // phase 2 operand: dO^T (dV) or Q^T (dK)
    if (tid < BK_Q) { Lbuf[PAR * BK_Q + tid] = st_l * LOG2E; Dlbuf[PAR * BK_Q + tid] = st_d; }
    // tile `it` is there for everyone, and everyone is done with tile it-1 and its P
    wait_async_tiles();
    __syncthreads();
    if (it + 1 < iters) fetch(it + 1, 1 - PAR);
    const int q0 = qstart + (it % nqt) * BK_Q;
    // phase 1: X[q, key] = rows(Q or dO) . (K or V)^T for both 32-query blocks
    f32x16 xacc[NQB];
#pragma unroll
    for (int qb = 0; qb < NQB; ++qb) xacc[qb] = f32x16{};
    {
      constexpr int NSTEP = NQB * KS, AHEAD = 2;
      bf16x8 fx[AHEAD + 1];
#pragma unroll
      for (int n = 0; n < AHEAD && n < NSTEP; ++n) fx[n] = frag_rows<DHL>(rows_src, (n / KS) * 32, n % KS, lane);
#pragma unroll
      for (int n = 0; n < NSTEP; ++n) {
        const int m = n + AHEAD;
        if (m < NSTEP) fx[m % (AHEAD + 1)] = frag_rows<DHL>(rows_src, (m / KS) * 32, m % KS, lane);
        xacc[n / KS] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[n % (AHEAD + 1)], kvf[n % KS], xacc[n / KS], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    bf16x8 op[NQB][2];                                  // B operands of phase 2: P (role 0) or dS (role 1)
    if (role == 0) {
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int qoff = qb * 32 + g * 8 + half * 4;
          const f32x4 l4 = *reinterpret_cast<const f32x4*>(Ls + qoff);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = g * 4 + e;
            float p = __builtin_amdgcn_exp2f(fmaf(xacc[qb][r], scale_log2, -l4[e]));
            if (MASKED) {
              const int qi = q0 + qoff + e;
              if (qi >= Lq || kpos >= L || (CAUSAL && kpos > qi)) p = 0.f;
            }
            xacc[qb][r] = p;
          }
        }
        op[qb][0] = acc_to_operand(xacc[qb], 0);
        op[qb][1] = acc_to_operand(xacc[qb], 1);
        *reinterpret_cast<bf16x8*>(my_p + (qb * 2 + 0) * 64 * 8) = op[qb][0];
        *reinterpret_cast<bf16x8*>(my_p + (qb * 2 + 1) * 64 * 8) = op[qb][1];
      }
    }
    __syncthreads();                                    // P of this step is in LDS
    if (role == 1) {
#pragma unroll
      for (int qb = 0; qb < NQB; ++qb) {
        const bf16x8 pa = *reinterpret_cast<const bf16x8*>(my_p + (qb * 2 + 0) * 64 * 8);
        const bf16x8 pb = *reinterpret_cast<const bf16x8*>(my_p + (qb * 2 + 1) * 64 * 8);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(Dl + qb * 32 + g * 8 + half * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = g * 4 + e;
            const float p = (float)(r < 8 ? pa[r] : pb[r - 8]);
            xacc[qb][r] = p * (xacc[qb][r] - d4[e]);
          }
        }
        op[qb][0] = acc_to_operand(xacc[qb], 0);
        op[qb][1] = acc_to_operand(xacc[qb], 1);
      }
    }
    // phase 2: acc^T[c, key] += cols(dO or Q)^T . (P or dS), transposed operands requested one pair ahead
    {
      constexpr int NSTEP = NQB * NB;
      bf16x8 fr[2][2];
      fr[0][0] = frag_cols<DHL>(cols_src, 0, 0, lane);
      fr[0][1] = frag_cols<DHL>(cols_src, 0, 16, lane);
#pragma unroll
      for (int n = 0; n < NSTEP; ++n) {
        const int qb = n / NB, j = n % NB, m = n + 1;
        if (m < NSTEP) {
          fr[m & 1][0] = frag_cols<DHL>(cols_src, (m % NB) * 32, (m / NB) * 32, lane);
          fr[m & 1][1] = frag_cols<DHL>(cols_src, (m % NB) * 32, (m / NB) * 32 + 16, lane);
        }
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n & 1][0], op[qb][0], acc[j], 0, 0, 0);
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[n & 1][1], op[qb][1], acc[j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  // which query tiles need the mask tests: as in the single-wavefront kernel, per 32-key block
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  auto step_of = [&](int it, bool masked) {
    if (it & 1) { if (masked) step(it, std::true_type{}, P1{}); else step(it, std::false_type{}, P1{}); }
    else { if (masked) step(it, std::true_type{}, P0{}); else step(it, std::false_type{}, P0{}); }
  };
  {
    // (one call site per copy of the step: with two the compiler stops inlining them)
    const bool all_masked = kb0 + BK_KEYS > L;
    const int n_front = CAUSAL ? min(nqt, (kb * 32 + 32 + BK_Q - 1) / BK_Q) : 0;
    const int n_whole = max(n_front, (Lq - qstart) % BK_Q ? nqt - 1 : nqt);
    for (int it = 0, t = 0; it < iters; ++it, t = (t + 1 == nqt ? 0 : t + 1))
      step_of(it, all_masked || t < n_front || t >= n_whole);
  }
  const float out_scale = role == 0 ? 1.0f : scale;     // dV as it is, dK times the softmax scale
  if (kpos < L && gsplit > 1) {
    const size_t plane = (size_t)Ttot * Hkv * DH;
    float* pp = part + ((size_t)gs * 2 + (role == 0 ? 1 : 0)) * plane + (size_t)(lo + kpos) * (Hkv * DH) + hk * DH;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        if (DH % 32 == 0 || j * 32 + g * 8 + half * 4 < DH)
          *reinterpret_cast<f32x4*>(pp + j * 32 + g * 8 + half * 4) =
              f32x4{acc[j][g * 4] * out_scale, acc[j][g * 4 + 1] * out_scale, acc[j][g * 4 + 2] * out_scale,
                    acc[j][g * 4 + 3] * out_scale};
  } else if (kpos < L) {
    bf16_t* pp = (role == 0 ? dv : dk) + (size_t)(lo + kpos) * ldd + hk * DH;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16_t)(acc[j][g * 4 + e] * out_scale);
        if (DH % 32 == 0 || j * 32 + g * 8 + half * 4 < DH)
          *reinterpret_cast<bf16x4*>(pp + j * 32 + g * 8 + half * 4) = w;
      }
  }
}

// dK, dV at head size 128 over many keys: the pair scheme with 64 keys per pair (256 per workgroup).
// Every Q / dO fragment read from LDS feeds two MFMAs instead of one, and a Q / dO tile is brought in
// for twice the keys: with 32 keys per pair the LDS pipe is busy as long as the matrix pipe (fragment
// reads, fills and the P exchange of a 32x32 block: about 1130 clocks of LDS for 1024 of MFMAs).
// 128 accumulator registers and 64 of K or V leave 64 for everything else, so
//  - a step is one 32-query block;
//  - tiles lie in LDS as RunTile has them, so that every read is one lane constant plus an immediate offset.
// Tiles go through a ring of four buffers, requested three steps ahead; one barrier per step hands over
// P and the next tile.
// Against 32 keys per pair, us: 8192 queries x 8192 keys, 32 / 8 heads, 2207 -> 1875 (1.17 PFLOP/s of MFMAs), causal
// 1138 -> 1002; 16 samples of about 1160 tokens, 24 heads, 848 -> 657; 8192 tokens of causal documents, 32
// heads, 435 -> 365.  Fragments requested three steps ahead and a raised wave priority around the MFMAs
// changed nothing.
struct WideTile {
  static constexpr int ROWS = 32, PART = RunTile<128>::bytes(ROWS);
  static constexpr int Q = 0, D = PART, LSE = 2 * PART, DELTA = LSE + ROWS * 4, BYTES = DELTA + ROWS * 4;
  static constexpr int RING = 4;
};

// the lane index, computed anew
__device__ inline int fresh_lane() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

constexpr int DKDV_WIDE_LDS_BYTES = WideTile::RING * WideTile::BYTES + 2 * 4 * 4096;
template <bool CAUSAL>
__device__ inline void dkdv_wide_tile(
    unsigned char* lds, int block, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cuq, const int32_t* __restrict__ cu,
    int S, bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int ldd, int Tq, int Ttot, int Hkv, int group,
    float scale, float scale_log2, int gsplit,
    float* __restrict__ part /* [gsplit][2][Ttot][Hkv*DH] fp32 when gsplit > 1 */, SeqOrder ord) {
  constexpr int DH = 128, KS = 8, NB = 4, KB = 2;
  using W = WideTile;
  using RT = RunTile<DH>;
  static_assert(W::RING * W::BYTES % 1024 == 0, "P starts where a tile run may");
  unsigned char* const tiles = lds;
  unsigned char* const Pbuf = lds + W::RING * W::BYTES;  // [parity][pair][key block, half k-step][lane]
  int seq, kt, nkt, tile_id, hk, hk_gs;
  tile_and_head(Hkv * gsplit, &tile_id, &hk_gs, block);
  hk = hk_gs / gsplit;
  const int gs = hk_gs % gsplit;
  const int gpart = group / gsplit;
  if (!find_tile(cu, ord, S, WIDE_KEYS, tile_id, &seq, &kt, &nkt)) return;
  kt = nkt - 1 - kt;                                   // early key tiles see the most queries
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  const int loq = cuq[seq], Lq = cuq[seq + 1] - loq;
  const int kb0 = kt * WIDE_KEYS;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pair = wave & 3;                            // wavefronts w and w+4 share a SIMD
  const int key0 = kb0 + pair * 64;                     // the pair's first key
  const int qstart = CAUSAL ? kb0 : 0;
  const int nqt = Lq > qstart ? (Lq - qstart + W::ROWS - 1) / W::ROWS : 0;   // no query: dk = dv = 0
  const int iters = nqt * gpart;
  const int head0 = hk * group + gs * gpart;
  // A pair needs the mask tests where its keys are cut by the sequence end, on the last query tile when that is
  // cut, and up to its last key under a causal mask; it sits out the query tiles before its first key,
  // and all of them if it lies past the sequence.
  const bool keys_cut = key0 + 64 > L;
  const int skip = key0 >= L ? nqt : CAUSAL ? min(nqt, (key0 - qstart) / W::ROWS) : 0;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)tiles;
  constexpr int LOADS = 3;

  // Everything of a role is compiled on its own: its registers are allocated for it alone.  Addresses are derived
  // from the lane index in every step; kept in registers, they would push K or V fragments out to memory.
  auto run = [&](auto role_t) {
    constexpr int ROLE = decltype(role_t)::value;
    constexpr int ROWS_AT = ROLE == 0 ? W::Q : W::D, COLS_AT = ROLE == 0 ? W::D : W::Q;
    constexpr int STATS_AT = ROLE == 0 ? W::LSE : W::DELTA;
    bf16x8 kvf[KB][KS];                                   // role 0 keeps K (for S), role 1 keeps V (for dP)
    {
      const int l = fresh_lane();
#pragma unroll
      for (int b = 0; b < KB; ++b) {
        const bf16_t* p = (ROLE == 0 ? k : v) + (size_t)(lo + min(key0 + b * 32 + (l & 31), L - 1)) * ldk + hk * DH;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kvf[b][ks] = load_chunk<DH>(p, ks * 2 + (l >> 5));
      }
    }
    f32x16 acc[NB][KB];                                   // role 0: dV^T, role 1: dK^T (unscaled)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int b = 0; b < KB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][b][r] = 0.f;

    // role 0's wavefronts bring in Q and lse, role 1's dO and delta: two runs and a quarter of the row
    // statistics each, three loads per wavefront and step
    const int sld = ROLE == 0 ? ld : ldo;
    const bf16_t* src = scalar_ptr((ROLE == 0 ? q : d_o) + ((size_t)loq + qstart) * sld + head0 * DH);
    const float* stat = reinterpret_cast<const float*>(scalar_ptr((ROLE == 0 ? lse : delta) + (size_t)head0 * Tq + loq + qstart));
    int fn = 0, ft = 0;                                   // next tile to request: step, query tile of its head
    auto fetch = [&] {
      if (fn >= iters) return;
      const int last = Lq - qstart - 1 - ft * W::ROWS;    // rows past the sequence are clamped: their P is 0
      const uint32_t dst = lds0 + (fn & (W::RING - 1)) * W::BYTES;
      const int l = fresh_lane();
      const int row = RT::load_row(l), chunk = RT::load_chunk(l) * 16;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = pair * 2 + i;
        const uint32_t off = (uint32_t)min(r * RT::RPR + row, last) * (uint32_t)sld * 2u + (uint32_t)chunk;
        TileAsync<32, DH, 256>::load16(src, off, dst + ROWS_AT + r * RT::RUN);
      }
      const uint32_t off = (uint32_t)min(pair * 8 + (l & 7), last) * 4u;
      if (l < 8)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                     :: "s"(dst + STATS_AT + pair * 32), "v"(off), "s"(stat) : "memory", "m0");
      ++fn;
      src += (size_t)W::ROWS * sld;
      stat += W::ROWS;
      if (++ft == nqt) {                                  // first query tile of the next head
        ft = 0;
        src += DH - (size_t)nqt * W::ROWS * sld;
        stat += Tq - (size_t)nqt * W::ROWS;
      }
    };
    auto tile_of = [&](int n) { return tiles + (n & (W::RING - 1)) * W::BYTES; };
    auto p_of = [&](int n) { return Pbuf + (n & 1) * (4 * 4096) + pair * 4096 + fresh_lane() * 16; };
    auto barrier = [] {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    // between the phases of step n: its P is in LDS, and the next step's tile; the one after may still be on its way
    auto hand_over = [&](int n) {
      if (n + 2 < iters) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((W::RING - 3) * LOADS) : "memory");
      else wait_async_tiles();
      barrier();
    };
    // phase 1: X[q, key] += rows(Q or dO) . (K or V)^T
    auto scores = [&](int n, f32x16 (&x)[KB]) {
      const unsigned char* rows = tile_of(n) + ROWS_AT + RT::rows_at(fresh_lane());
      constexpr int AHEAD = 2;
      bf16x8 fx[AHEAD + 1];
      auto request = [&](int ks) { fx[ks % (AHEAD + 1)] = RT::read_rows(rows, 0, ks); };
#pragma unroll
      for (int ks = 0; ks < AHEAD; ++ks) request(ks);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + AHEAD < KS) request(ks + AHEAD);
#pragma unroll
        for (int b = 0; b < KB; ++b)
          x[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[ks % (AHEAD + 1)], kvf[b][ks], x[b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // phase 2: acc^T[c, key] += cols(dO or Q)^T . (P or dS), transposed operands requested ahead
    auto accumulate = [&](int n, const bf16x8 (&op)[KB][2]) {
      const unsigned char* cols = tile_of(n) + COLS_AT + RT::cols_at(fresh_lane());
      auto request = [&](int m) { return RT::read_cols(cols, m >> 1, m & 1); };   // m = j * 2 + t: 32 columns of dh, 16 query rows
      constexpr int AHEAD = 2;
      bf16x8 fc[AHEAD + 1];
#pragma unroll
      for (int m = 0; m < AHEAD; ++m) fc[m] = request(m);
      if (ROLE == 0) fetch();                              // step n + 3, over the tile of step n - 1
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int m = 0; m < NB * 2; ++m) {
        if (m + AHEAD < NB * 2) fc[(m + AHEAD) % (AHEAD + 1)] = request(m + AHEAD);
#pragma unroll
        for (int b = 0; b < KB; ++b)
          acc[m >> 1][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fc[m % (AHEAD + 1)], op[b][m & 1], acc[m >> 1][b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto step = [&](int n, int q0) {
      // accumulator element (g, b, e) of a lane: query q0 + 4 half + (8 g + e), key key0 + lane % 32 + 32 b
      f32x16 x[KB];
      bf16x8 op[KB][2];
      if constexpr (ROLE == 0) {
        x[0] = x[1] = f32x16{};
        scores(n, x);
        if (keys_cut || q0 + W::ROWS > Lq || (CAUSAL && q0 < key0 + 63)) {
          asm volatile("");                                 // keeps the tests out of the steps that need none
          const int l = fresh_lane(), h4 = (l >> 5) * 4, ki = key0 + (l & 31);
          const int q_left = Lq - q0 - h4, k_left = L - ki, ahead = ki - q0 - h4;
#pragma unroll
          for (int g = 0; g < 4; ++g)
#pragma unroll
            for (int b = 0; b < KB; ++b)
#pragma unroll
              for (int e = 0; e < 4; ++e)
                if (q_left <= g * 8 + e || k_left <= b * 32 || (CAUSAL && ahead > g * 8 + e - b * 32))
                  x[b][g * 4 + e] = -INFINITY;              // P = 0
        }
        const unsigned char* stats = tile_of(n) + STATS_AT + (fresh_lane() >> 5) * 16;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 l4 = *reinterpret_cast<const f32x4*>(stats + g * 32) * LOG2E;
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              x[b][g * 4 + e] = __builtin_amdgcn_exp2f(fmaf(x[b][g * 4 + e], scale_log2, -l4[e]));
        }
        unsigned char* my_p = p_of(n);
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            op[b][t] = acc_to_operand(x[b], t);
            *reinterpret_cast<bf16x8*>(my_p + (b * 2 + t) * 1024) = op[b][t];
          }
        hand_over(n);
      } else {
        x[0] = x[1] = f32x16{};
        scores(n, x);
        // dP - delta while the partner takes its exponentials (dP that starts at -delta saves the subtractions and
        // 2 % of the kernel, and rounds some sums differently)
        const unsigned char* stats = tile_of(n) + STATS_AT + (fresh_lane() >> 5) * 16;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 d4 = *reinterpret_cast<const f32x4*>(stats + g * 32);
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[b][g * 4 + e] -= d4[e];
        }
        asm volatile("" : "+v"(x[0]), "+v"(x[1]));          // (subtracted here: behind the barrier, delta would push V fragments out)
        hand_over(n);
        const unsigned char* my_p = p_of(n);
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
          for (int t = 0; t < 2; ++t) op[b][t] = *reinterpret_cast<const bf16x8*>(my_p + (b * 2 + t) * 1024);
        fetch();                                           // step n + 3, over the tile of step n - 1
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int b = 0; b < KB; ++b)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int e = 0; e < 8; ++e) x[b][t * 8 + e] *= (float)op[b][t][e];
            op[b][t] = acc_to_operand(x[b], t);
          }
      }
      accumulate(n, op);
    };

    settle_compiler_loads();                              // K / V fragments, offsets
    for (int n = 0; n < W::RING - 1; ++n) fetch();
    if (iters > W::RING - 2) asm volatile("s_waitcnt vmcnt(%0)" :: "n"((W::RING - 2) * LOADS) : "memory");
    else wait_async_tiles();
    barrier();
    for (int n = 0; n < iters;) {
      for (int t = 0; t < skip; ++t, ++n) { hand_over(n); fetch(); }
      for (int t = skip; t < nqt; ++t, ++n) step(n, qstart + t * W::ROWS);
    }

    const float out_scale = ROLE == 0 ? 1.0f : scale;     // dV as it is, dK times the softmax scale
    const int l = fresh_lane();
#pragma unroll
    for (int b = 0; b < KB; ++b) {
      const int key = key0 + b * 32 + (l & 31);
      if (key >= L) continue;
      const size_t row = (size_t)(lo + key);
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const int c = hk * DH + j * 32 + g * 8 + (l >> 5) * 4;
          f32x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = acc[j][b][g * 4 + e] * out_scale;
          if (gsplit > 1) {
            *reinterpret_cast<f32x4*>(part + ((size_t)gs * 2 + (ROLE == 0 ? 1 : 0)) * Ttot * Hkv * DH + row * (Hkv * DH) + c) = w;
          } else {
            bf16x4 h;
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = (bf16_t)w[e];
            *reinterpret_cast<bf16x4*>((ROLE == 0 ? dv : dk) + row * ldd + c) = h;
          }
        }
    }
  };
  if (wave < 4) run(std::integral_constant<int, 0>{});
  else run(std::integral_constant<int, 1>{});
}

// dQ of one 128-row query tile of one q head: walks the key tiles, scores kept as
// S^T[key, q] as in the forward kernel.
template <int DH> constexpr int dq_lds_bytes() { return 4 * (DH > 72 ? 32 : FK) * HeadDim<DH>::DHL * 2; }
template <int DH, bool CAUSAL>
__device__ inline void dq_tile(unsigned char* lds, int tid, int tile_id, int hq, bool live, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk,
    int S, bf16_t* __restrict__ dq, int ldd, int Ttot, int group, float scale, float scale_log2,
    SeqOrder ord) {
  // K and V tiles are double-buffered and streamed into LDS as in the forward kernel; Q and dO of
  // this wavefront's 32 queries stay in registers.  At head size 128 a step is one 32-key block:
  // with two blocks' fragments and masks in flight next to Q, dO and the dQ accumulator the
  // kernel spills at two wavefronts per SIMD.  (dO read from LDS instead, a quarter more fragment
  // reads per key block, measured 1 % slower.)
  constexpr int FKD = DH > 72 ? 32 : FK;
  constexpr int TILE = FKD * HeadDim<DH>::DHL;
  bf16_t* const Kbuf = reinterpret_cast<bf16_t*>(lds);
  bf16_t* const Vbuf = Kbuf + 2 * TILE;
  int seq, qt, nqt;
  if (!find_tile(cu, ord, S, FQ, tile_id, &seq, &qt, &nqt)) return;
  const int hk = hq / group;
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  const int lok = cuk[seq], Lk = cuk[seq + 1] - lok;
  const int q0 = qt * FQ;
  const int lane = tid & 63, wave = tid >> 6, half = lane >> 5;
  const int qpos = q0 + wave * 32 + (lane & 31);
  const int qrow = min(qpos, L - 1);
  if (Lk == 0) {
    // no key in this chunk (workgroup-uniform): dq = 0
    if (live && qpos < L) {
      bf16_t* pq = dq + (size_t)(lo + qpos) * ldd + hq * DH;
      for (int c = half * (DH / 2); c < (half + 1) * (DH / 2); c += 4) {
        bf16x4 z = {(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
        *reinterpret_cast<bf16x4*>(pq + c) = z;
      }
    }
    return;
  }

  bf16x8 qf[HeadDim<DH>::KS], dof[HeadDim<DH>::KS];
  {
    const bf16_t* qp = q + (size_t)(lo + qrow) * ld + hq * DH;
    const bf16_t* dp = d_o + (size_t)(lo + qrow) * ldo + hq * DH;
#pragma unroll
    for (int ks = 0; ks < HeadDim<DH>::KS; ++ks) {
      qf[ks] = load_chunk<DH>(qp, ks * 2 + half);
      dof[ks] = load_chunk<DH>(dp, ks * 2 + half);
    }
  }
  const float my_lse = lse[(size_t)hq * Ttot + lo + qrow] * LOG2E;
  const float my_delta = delta[(size_t)hq * Ttot + lo + qrow];
  f32x16 dqacc[HeadDim<DH>::NB];
#pragma unroll
  for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) dqacc[j][r] = 0.f;

  const int kend = CAUSAL ? min(Lk, q0 + FQ) : Lk;
  const int nkt = (kend + FKD - 1) / FKD;
  const bf16_t* kbase = k + (size_t)lok * ldk + hk * DH;
  const bf16_t* vbase = v + (size_t)lok * ldk + hk * DH;
  using Tile = TileAsync<FKD, DH, 256>;
  Tile tile;
  tile.init(ldk, tid);
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    Tile::zero_padding(Kbuf + b * TILE, tid);
    Tile::zero_padding(Vbuf + b * TILE, tid);
  }
  tile.issue(kbase, ldk, Lk, Kbuf, wave_u);
  tile.issue(vbase, ldk, Lk, Vbuf, wave_u);
  settle_compiler_loads();                 // the Q and dO fragments, lse, delta (and, with them, tile 0)
  // two copies of the step, without and with the mask test, as in the forward kernel
  constexpr bool FOLD_DELTA = DH <= 64;      // dP accumulators start at -delta: the MFMAs leave dP - delta
  f32x16 dp_start = {};
  if (FOLD_DELTA)
#pragma unroll
    for (int r = 0; r < 16; ++r) dp_start[r] = -my_delta;
  auto step = [&](int kt, auto masked, auto parity) {
    constexpr bool MASKED = decltype(masked)::value;
    constexpr int PAR = decltype(parity)::value;
    const bf16_t* Ks = Kbuf + PAR * TILE;
    const bf16_t* Vs = Vbuf + PAR * TILE;
    wait_async_tiles();
    __syncthreads();      // tile kt is there for everyone, and everyone is done with tile kt-1
    if (kt + 1 < nkt) {
      const size_t next = (size_t)(kt + 1) * FKD * ldk;
      tile.issue(kbase + next, ldk, Lk - (kt + 1) * FKD, Kbuf + (1 - PAR) * TILE, wave_u);
      tile.issue(vbase + next, ldk, Lk - (kt + 1) * FKD, Vbuf + (1 - PAR) * TILE, wave_u);
    }
    const int key0 = kt * FKD;
    // S^T = K Q^T and dP^T = V dO^T of BP 32-key blocks are issued before any softmax arithmetic,
    // so that one block's MFMAs run under the other's vector work; at head size 128 that is one
    // block at a time (two sets of accumulators do not fit next to two resident wavefronts).
    constexpr int NBLK = FKD / 32, BP = DH > 72 ? 1 : NBLK, KS = HeadDim<DH>::KS;
#pragma unroll
    for (int b0 = 0; b0 < NBLK; b0 += BP) {
      f32x16 sacc[BP], dpacc[BP];
#pragma unroll
      for (int bi = 0; bi < BP; ++bi) { sacc[bi] = f32x16{}; dpacc[bi] = dp_start; }
      {
        // operand fragments are requested AHEAD MFMA pairs before their use (see the dK/dV kernel)
        constexpr int NSTEP = BP * KS, AHEAD = 2;
        bf16x8 fk[AHEAD + 1], fv[AHEAD + 1];
        auto request = [&](int n) {
          fk[n % (AHEAD + 1)] = frag_rows<HeadDim<DH>::DHL>(Ks, (b0 + n / KS) * 32, n % KS, lane);
          fv[n % (AHEAD + 1)] = frag_rows<HeadDim<DH>::DHL>(Vs, (b0 + n / KS) * 32, n % KS, lane);
        };
#pragma unroll
        for (int n = 0; n < AHEAD && n < NSTEP; ++n) request(n);
#pragma unroll
        for (int n = 0; n < NSTEP; ++n) {
          const int bi = n / KS, ks = n % KS;
          if (n + AHEAD < NSTEP) request(n + AHEAD);
          sacc[bi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[n % (AHEAD + 1)], qf[ks], sacc[bi], 0, 0, 0);
          dpacc[bi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[n % (AHEAD + 1)], dof[ks],
                                                              dpacc[bi], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int bi = 0; bi < BP; ++bi) {
        const int b = b0 + bi;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float p = __builtin_amdgcn_exp2f(fmaf(sacc[bi][r], scale_log2, -my_lse));
          if (MASKED) {
            const int key = key0 + b * 32 + (r >> 2) * 8 + half * 4 + (r & 3);
            if (key >= Lk || (CAUSAL && key > qpos)) p = 0.f;
          }
          dpacc[bi][r] = FOLD_DELTA ? p * dpacc[bi][r] : p * (dpacc[bi][r] - my_delta);
        }
        const bf16x8 s0 = acc_to_operand(dpacc[bi], 0), s1 = acc_to_operand(dpacc[bi], 1);
        {
          // dQ += dS K, the transposed K operands requested one pair of MFMAs ahead
          constexpr int NB = HeadDim<DH>::NB;
          bf16x8 fr[2][2];
          fr[0][0] = frag_cols<HeadDim<DH>::DHL>(Ks, 0, b * 32, lane);
          fr[0][1] = frag_cols<HeadDim<DH>::DHL>(Ks, 0, b * 32 + 16, lane);
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if (j + 1 < NB) {
              fr[(j + 1) & 1][0] = frag_cols<HeadDim<DH>::DHL>(Ks, (j + 1) * 32, b * 32, lane);
              fr[(j + 1) & 1][1] = frag_cols<HeadDim<DH>::DHL>(Ks, (j + 1) * 32, b * 32 + 16, lane);
            }
            dqacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][0], s0, dqacc[j], 0, 0, 0);
            dqacc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[j & 1][1], s1, dqacc[j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  };
  int n_plain = Lk / FKD;
  if (CAUSAL) n_plain = min(n_plain, (q0 + wave * 32 + 1) / FKD);
  n_plain = min(n_plain, nkt);
  using P0 = std::integral_constant<int, 0>;
  using P1 = std::integral_constant<int, 1>;
  for (int kt = 0; kt < nkt; ++kt) {
    const bool plain = kt < n_plain;
    if (kt & 1) { if (plain) step(kt, std::false_type{}, P1{}); else step(kt, std::true_type{}, P1{}); }
    else { if (plain) step(kt, std::false_type{}, P0{}); else step(kt, std::true_type{}, P0{}); }
  }
  if (live && qpos < L) {
    bf16_t* pq = dq + (size_t)(lo + qpos) * ldd + hq * DH;
#pragma unroll
    for (int j = 0; j < HeadDim<DH>::NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16_t)(dqacc[j][g * 4 + e] * scale);
        if (DH % 32 == 0 || j * 32 + g * 8 + half * 4 < DH)
          *reinterpret_cast<bf16x4*>(pq + j * 32 + g * 8 + half * 4) = w;
      }
  }
}

// head sizes above 64, two workgroups per CU: packs whose dK/dV tiles alone fill the chip (see bwd_plan)
template <int DH, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void fa_bwd_dq_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk,
    int S, bf16_t* __restrict__ dq, int ldd, int Ttot, int Hq, int group, float scale, float scale_log2,
    SeqOrder ord) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[dq_lds_bytes<DH>()];
  int tile, head;
  tile_and_head(Hq, &tile, &head, blockIdx.x);
  dq_tile<DH, CAUSAL>(lds, threadIdx.x, tile, head, true, q, k, v, ld, ldk, d_o, ldo, lse, delta, cu, cuk, S, dq, ldd, Ttot,
                      group, scale, scale_log2, ord);
}

// The whole backward of head size 64 behind delta in one grid: the dK/dV tiles, which run longer, then the dQ tiles, which
// fill the CUs that the last of them leave.  Both have two wavefronts per SIMD.  They share one piece of LDS (with one
// each the dK/dV tile spills).  16 heads, two launches -> one: 577 tokens 41 -> 26 us, 6 images 47 -> 34, 26 images 236 -> 223, 8192
// tokens 985 -> 970; causal 41 -> 26, 45 -> 31, 179 -> 165, 547 -> 507.
template <int DH, bool CAUSAL>
__global__ __launch_bounds__(256, 2) void fa_bwd_joint_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld, int ldk,
    const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse, const float* __restrict__ delta,
    const int32_t* __restrict__ cuq, const int32_t* __restrict__ cuk, int S, bf16_t* __restrict__ dq, int ldd,
    bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int ldd_kv, int Tq, int Tk, int Hkv, int group, float scale,
    float scale_log2, int gsplit, float* __restrict__ part, int kv_wgs, SeqOrder ord_kv, SeqOrder ord_q) {
  constexpr int LDS = dkdv_lds_bytes<DH>() > dq_lds_bytes<DH>() ? dkdv_lds_bytes<DH>() : dq_lds_bytes<DH>();
  __shared__ __attribute__((aligned(1024))) unsigned char lds[LDS];
  if ((int)blockIdx.x < kv_wgs)
    dkdv_tile<DH, CAUSAL>(lds, blockIdx.x, q, k, v, ld, ldk, d_o, ldo, lse, delta, cuq, cuk, S, dk, dv, ldd_kv, Tq, Tk, Hkv,
                          group, scale, scale_log2, gsplit, part, ord_kv);
  else
  {
    int tile, head;
    tile_and_head(Hkv * group, &tile, &head, blockIdx.x - kv_wgs);
    dq_tile<DH, CAUSAL>(lds, threadIdx.x, tile, head, true, q, k, v, ld, ldk, d_o, ldo, lse, delta, cuq, cuk, S, dq, ldd, Tq,
                        group, scale, scale_log2, ord_q);
  }
}

// dQ with two groups of wavefronts that take turns (see the forward kernel): while one multiplies -- dS K of a key
// tile, then Q K and dO V of the next -- the other one turns its scores into dS.  At head size 64, where the
// MFMAs of a tile are no longer than its softmax, the kernel above is ahead (96 against 112 us on 16384 tokens of images).
// us, two workgroups of four wavefronts -> this: 8192 x 8192 keys, 32 / 8 heads, 1522 -> 1332, causal 782 -> 687; 32768 tokens
// of causal documents 4217 -> 3630; 8192 tokens of documents, 32 heads, 262 -> 253; 16 samples of about 1130, 24 heads, 445 both.
constexpr int DQ_ALT_LDS_BYTES = (4 + 3) * RunTile<128>::bytes(FK);
template <bool CAUSAL>
__device__ inline void dq_alt_tile(
    unsigned char* lds, int block, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld,
    int ldk, const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse,
    const float* __restrict__ delta, const int32_t* __restrict__ cu, const int32_t* __restrict__ cuk,
    int S, bf16_t* __restrict__ dq, int ldd, int Ttot, int Hq, int group, float scale, float scale_log2,
    SeqOrder ord) {
  constexpr int DH = 128;
  using RT = RunTile<DH>;
  constexpr int KS = DH / 16, NB = DH / 32, KBL = FK / 32, TILE = RT::bytes(FK), RUNS = FK / RT::RPR / 8;
  constexpr int KRING = 4, VRING = 3;                     // a K tile is read as rows in one phase, as columns two later
  static_assert((KRING + VRING) * TILE == DQ_ALT_LDS_BYTES && TILE % 16 == 0, "the caller's piece of LDS");
  unsigned char* const Kbuf = lds;
  unsigned char* const Vbuf = lds + KRING * TILE;
  int seq, qt, nqt, tile_id, hq;
  tile_and_head(Hq, &tile_id, &hq, block);
  if (!find_tile(cu, ord, S, AQ, tile_id, &seq, &qt, &nqt)) return;
  const int hk = hq / group;
  const int lo = cu[seq], L = cu[seq + 1] - lo;
  const int lok = cuk[seq], Lk = cuk[seq + 1] - lok;
  const int q0 = qt * AQ;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qfirst = q0 + wave * 32;
  const int qpos = qfirst + (lane & 31);                  // this lane's query (column of S^T)
  const int qrow = min(qpos, L - 1);
  bf16x8 qf[KS], dof[KS];
  {
    const bf16_t* qp = q + (size_t)(lo + qrow) * ld + hq * DH;
    const bf16_t* dp = d_o + (size_t)(lo + qrow) * ldo + hq * DH;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qf[ks] = load_chunk<DH>(qp, ks * 2 + half);
      dof[ks] = load_chunk<DH>(dp, ks * 2 + half);
    }
  }
  const float my_lse = lse[(size_t)hq * Ttot + lo + qrow] * LOG2E;
  const float my_delta = delta[(size_t)hq * Ttot + lo + qrow];
  f32x16 dqacc[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) dqacc[j] = f32x16{};
  // key tiles of the workgroup, and those of this wavefront (none if its queries lie past the sequence)
  const int nkt = ((CAUSAL ? min(Lk, q0 + AQ) : Lk) + FK - 1) / FK;
  const int mine = qfirst >= L ? 0 : CAUSAL ? min(nkt, (qfirst + 31) / FK + 1) : nkt;
  const int plain = CAUSAL ? min(Lk / FK, (qfirst + 1) / FK) : Lk / FK;   // leading tiles that need no mask test
  const bf16_t* kbase = scalar_ptr(k + (size_t)lok * ldk + hk * DH);
  const bf16_t* vbase = scalar_ptr(v + (size_t)lok * ldk + hk * DH);
  const uint32_t klds = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)Kbuf;
  const uint32_t vlds = (uint32_t)(size_t)(__attribute__((address_space(3))) unsigned char*)Vbuf;
  // tile t of K or V into a ring slot; rows past the keys are clamped (their dS is 0)
  auto fetch = [&](const bf16_t* base, uint32_t dst, int t) {
    if (t >= nkt) return;
    const int l = fresh_lane();
    const bf16_t* src = base + (size_t)t * FK * ldk;
    const int last = Lk - t * FK - 1;
#pragma unroll
    for (int i = 0; i < RUNS; ++i) {
      const int r = wave * RUNS + i;
      const uint32_t off = (uint32_t)min(r * RT::RPR + RT::load_row(l), last) * (uint32_t)ldk * 2u + (uint32_t)RT::load_chunk(l) * 16u;
      TileAsync<FK, DH, 512>::load16(src, off, dst + r * RT::RUN);
    }
  };
  f32x16 sacc[KBL], dpacc[KBL];
  bf16x8 ds[KBL][2];
  auto scores = [&](int kslot, int vslot) {               // S^T = K Q^T, dP^T = V dO^T of a key tile
    const int at = RT::rows_at(fresh_lane());
    int ka = kslot * TILE + at, va = vslot * TILE + at;
    asm volatile("" : "+v"(ka), "+v"(va));                 // one register each; the rest is immediates
    constexpr int NSTEP = KBL * KS, AHEAD = 2;             // step n: key block n % KBL, k-step n / KBL
    bf16x8 fk[AHEAD + 1], fv[AHEAD + 1];
    auto request = [&](int n) {
      fk[n % (AHEAD + 1)] = RT::read_rows(Kbuf + ka, n % KBL, n / KBL);
      fv[n % (AHEAD + 1)] = RT::read_rows(Vbuf + va, n % KBL, n / KBL);
    };
#pragma unroll
    for (int b = 0; b < KBL; ++b) sacc[b] = dpacc[b] = f32x16{};
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) request(n);
#pragma unroll
    for (int n = 0; n < NSTEP; ++n) {
      if (n + AHEAD < NSTEP) request(n + AHEAD);
      sacc[n % KBL] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk[n % (AHEAD + 1)], qf[n / KBL], sacc[n % KBL], 0, 0, 0);
      dpacc[n % KBL] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fv[n % (AHEAD + 1)], dof[n / KBL], dpacc[n % KBL], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto accumulate = [&](int kslot) {                      // dQ^T += K^T dS^T
    int at = kslot * TILE + RT::cols_at(fresh_lane());
    asm volatile("" : "+v"(at));
    constexpr int NSTEP = KBL * 2 * NB, AHEAD = 3;         // step n: 16 keys n / NB, 32 columns n % NB
    bf16x8 f[AHEAD + 1];
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) f[n] = RT::read_cols(Kbuf + at, n % NB, n / NB);
#pragma unroll
    for (int n = 0; n < NSTEP; ++n) {
      if (n + AHEAD < NSTEP) f[(n + AHEAD) % (AHEAD + 1)] = RT::read_cols(Kbuf + at, (n + AHEAD) % NB, (n + AHEAD) / NB);
      dqacc[n % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f[n % (AHEAD + 1)], ds[n / NB / 2][n / NB % 2], dqacc[n % NB], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto softmax = [&](int t) {
    if (t >= plain) {
      asm volatile("");                                    // keeps the tests out of the tiles that need none
      const int h4 = (fresh_lane() >> 5) * 4, left = Lk - t * FK - h4, ahead = qfirst + (fresh_lane() & 31) - t * FK - h4;
#pragma unroll
      for (int b = 0; b < KBL; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int e = b * 32 + (r >> 2) * 8 + (r & 3);
          if (e >= left || (CAUSAL && e > ahead)) sacc[b][r] = -INFINITY;   // P = 0
        }
    }
#pragma unroll
    for (int b = 0; b < KBL; ++b) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sacc[b][r], scale_log2, -my_lse));
        dpacc[b][r] = p * (dpacc[b][r] - my_delta);
      }
      ds[b][0] = acc_to_operand(dpacc[b], 0);
      ds[b][1] = acc_to_operand(dpacc[b], 1);
    }
  };
  settle_compiler_loads();                                // Q and dO fragments, lse, delta, offsets
  fetch(kbase, klds, 0);
  fetch(vbase, vlds, 0);
  fetch(kbase, klds + TILE, 1);
  fetch(vbase, vlds + TILE, 1);
  wait_async_tiles();
  phase_barrier();
  if (wave >= 4) phase_barrier();                         // the second group stays one phase behind
  if (mine > 0) scores(0, 0);
  phase_barrier();
  for (int t = 0, v1 = 1, v2 = 2; t < nkt; ++t) {         // V slots of tiles t + 1, t + 2
    // both groups are past the tiles these overwrite (K t - 2, V t - 1); they are read two phases from now
    fetch(kbase, klds + ((t + 2) & (KRING - 1)) * TILE, t + 2);
    fetch(vbase, vlds + v2 * TILE, t + 2);
    if (t < mine) softmax(t);
    phase_barrier();
    if (t < mine) accumulate(t & (KRING - 1));
    if (t + 1 < mine) scores((t + 1) & (KRING - 1), v1);
    wait_async_tiles();
    phase_barrier();
    v1 = v2;
    v2 = v2 == VRING - 1 ? 0 : v2 + 1;
  }
  if (wave < 4) phase_barrier();
  if (qpos < L) {
    bf16_t* pq = dq + (size_t)(lo + qpos) * ldd + hq * DH;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        bf16x4 w;
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] = (bf16_t)(dqacc[j][g * 4 + e] * scale);
        *reinterpret_cast<bf16x4*>(pq + j * 32 + g * 8 + half * 4) = w;
      }
  }
}

// ... and of the head sizes above 64, in workgroups of eight wavefronts: dK/dV by pairs of wavefronts (WIDE: with 64 keys a
// pair), dQ with turns (ALT) or as the 128 rows of two heads side by side -- the same sequence and tile, so that both
// halves of the workgroup make the same steps and meet at the same barriers; with an odd number of heads the last
// workgroup's second half repeats the first and stores nothing.  Two launches -> one, us: 32 heads, 300 tokens 39 -> 27, causal
// documents of 8192 tokens 561 -> 534; 32 / 8 heads, 777 causal tokens 76 -> 55, 39000 tokens of heavy-tailed documents 9349 -> 8839;
// 16 two-stream samples of 1170 tokens, 24 heads, 1104 -> 1028.  The kernels with turns hold more than the 102 scalar registers there
// are (5 to 16 spill into lanes of a vector register; apart, dQ spilled two).
template <int DH, bool CAUSAL, bool WIDE, bool ALT>
__global__ __launch_bounds__(512, 2) void fa_bwd_joint512_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, int ld, int ldk,
    const bf16_t* __restrict__ d_o, int ldo, const float* __restrict__ lse, const float* __restrict__ delta,
    const int32_t* __restrict__ cuq, const int32_t* __restrict__ cuk, int S, bf16_t* __restrict__ dq, int ldd,
    bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int ldd_kv, int Tq, int Tk, int Hkv, int group, float scale,
    float scale_log2, int gsplit, float* __restrict__ part, int kv_wgs, SeqOrder ord_kv, SeqOrder ord_q) {
  constexpr int KV = WIDE ? DKDV_WIDE_LDS_BYTES : dkdv_pair_lds_bytes<DH>(), Q = ALT ? DQ_ALT_LDS_BYTES : 2 * dq_lds_bytes<DH>();
  __shared__ __attribute__((aligned(1024))) unsigned char lds[KV > Q ? KV : Q];
  const int Hq = Hkv * group;
  if ((int)blockIdx.x < kv_wgs) {
    if constexpr (WIDE)
      dkdv_wide_tile<CAUSAL>(lds, blockIdx.x, q, k, v, ld, ldk, d_o, ldo, lse, delta, cuq, cuk, S, dk, dv, ldd_kv, Tq, Tk, Hkv,
                             group, scale, scale_log2, gsplit, part, ord_kv);
    else
      dkdv_pair_tile<DH, CAUSAL>(lds, blockIdx.x, q, k, v, ld, ldk, d_o, ldo, lse, delta, cuq, cuk, S, dk, dv, ldd_kv, Tq, Tk,
                                 Hkv, group, scale, scale_log2, gsplit, part, ord_kv);
  } else if constexpr (ALT) {
    dq_alt_tile<CAUSAL>(lds, blockIdx.x - kv_wgs, q, k, v, ld, ldk, d_o, ldo, lse, delta, cuq, cuk, S, dq, ldd, Tq, Hq, group,
                        scale, scale_log2, ord_q);
  } else {
    int tile, heads;
    tile_and_head((Hq + 1) / 2, &tile, &heads, blockIdx.x - kv_wgs);
    const int side = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), head = heads * 2 + side;
    dq_tile<DH, CAUSAL>(lds + side * dq_lds_bytes<DH>(), threadIdx.x & 255, tile, min(head, Hq - 1), head < Hq, q, k, v, ld, ldk,
                        d_o, ldo, lse, delta, cuq, cuk, S, dq, ldd, Tq, group, scale, scale_log2, ord_q);
  }
}

// dk, dv = sum over the q-head parts of the fp32 partials, in part order
__global__ void fa_dkdv_reduce_kernel(const float* __restrict__ part, int gsplit, int Ttot, int W /* Hkv*dh */,
                                      bf16_t* __restrict__ dk, bf16_t* __restrict__ dv, int ldd) {
  const long i = ((long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
  const long plane = (long)Ttot * W;
  if (i >= plane) return;
  const int t = (int)(i / W), c = (int)(i % W);
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    for (int g = 0; g < gsplit; ++g) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(part + ((size_t)g * 2 + which) * plane + i);
      s[0] += v[0]; s[1] += v[1]; s[2] += v[2]; s[3] += v[3];
    }
    bf16x4 w = {(bf16_t)s[0], (bf16_t)s[1], (bf16_t)s[2], (bf16_t)s[3]};
    *reinterpret_cast<bf16x4*>((which == 0 ? dk : dv) + (size_t)t * ldd + c) = w;
  }
}

// q-head parts per kv head in the dK/dV kernel: more workgroups when few key tiles x kv
// heads would leave most CUs idle (grouped-query attention over a short pack)
int dkdv_group_split(int tiles, int Hkv, int group) {
  const long wgs = (long)tiles * Hkv;
  int want = (int)((1024 + wgs - 1) / wgs);
  int gsplit = 1;
  for (int s = 1; s <= group; ++s)
    if (group % s == 0 && s <= want) gsplit = s;
  return gsplit;
}

// The wide dK/dV kernel (head size 128) or the one with 128 keys per workgroup?  Both hold a CU alone.  Whole
// backward, us, narrow -> wide.  The wide one needs
//  - sequences that 256-key tiles cut about as well: 32 x 257, 16 heads, 168 -> 190;
//  - three workgroups per CU to even out its tiles (8 documents of 411 to 1800, 32 heads, 473 -> 431; 777 tokens, 32 heads, 70 ->
//    88), or, when all tiles take equally long, to be done in one round where the other is not: bidirectional 4 x 400,
//    24 heads, 85 -> 71; under a causal mask the longest tile decides: 4096, 16 heads, 297 -> 360; 2048 + 900 + two short, 16
//    heads, 145 -> 187;
//  - heads of a group that it splits no further than the other, or enough queries per key to pay for the fp32 partials:
//    32 / 8 heads, bidirectional, 24 x 256 (split 4 against 2), 193 -> 243; 12 x 640 403 -> 465; 16 x 1152 1398 -> 1371;
//    causal 4 x 2048 618 -> 639.  dK/dV alone of 8192 x 8192 keys 2207 -> 1875, causal 1138 -> 1002.
bool dkdv_wide(const AttnArgs& a) {
  const int tw = count_tiles(a.kv_cu_host(), a.S, WIDE_KEYS), tn = count_tiles(a.kv_cu_host(), a.S, BK_KEYS);
  if (tw == 0 || tw * 2L * 4 > tn * 5L) return false;
  const int group = a.Hq / a.Hkv, split_w = dkdv_group_split(tw, a.Hkv, group), split_n = dkdv_group_split(tn, a.Hkv, group);
  if (split_w != split_n && keys_per_query(a) < (a.causal ? 3000 : 1100)) return false;
  const long wide = (long)tw * a.Hkv * split_w, narrow = (long)tn * a.Hkv * split_n;
  return wide >= 3 * NUM_CU || (!a.causal && wide <= NUM_CU && narrow > NUM_CU);
}

// What a backward pass launches behind delta: tiles, workgroups, and whether dK/dV and dQ share a grid.
struct BwdPlan { bool wide, alt, together; int key_rows, query_rows, gsplit, kv_wgs, qtiles, q_wgs; };

BwdPlan bwd_plan(const AttnArgs& a) {
  BwdPlan p;
  p.wide = a.dh == 128 && dkdv_wide(a);
  p.alt = a.dh == 128 && queries_alternating(a);
  p.key_rows = p.wide ? WIDE_KEYS : BK_KEYS;
  p.query_rows = p.alt ? AQ : FQ;
  const int ktiles = count_tiles(a.kv_cu_host(), a.S, p.key_rows);
  p.gsplit = ktiles > 0 ? dkdv_group_split(ktiles, a.Hkv, a.Hq / a.Hkv) : 1;
  p.kv_wgs = ktiles * a.Hkv * p.gsplit;
  p.qtiles = count_tiles(a.cu_host, a.S, p.query_rows);
  const bool same_wgs = a.dh <= 64 || p.alt;              // dQ takes the workgroups of dK/dV
  p.q_wgs = p.qtiles * (same_wgs ? a.Hq : (a.Hq + 1) / 2);
  // One launch or two?  One, where dQ takes the same workgroups anyway: head size 64, and 256-row query tiles (60 packs of
  // 1500 to 36000 tokens: 57 faster, 3 % on average, 12 % at best, the slowest -1.6 %).  Where both parts fill whole rounds there is nothing to
  // gain: 32 / 8 heads, 8192 queries and keys 3217 -> 3172, causal 1729 -> 1733; the four pairs of a rank 14668 -> 14612, in eight runs +1.0 %
  // to -0.8 %.  The 128 rows of two heads side by
  // side are slower than two workgroups on a CU, so that is for packs whose workgroups all run at once, or nearly so where a
  // causal mask makes most of them short or the wide dK/dV ones are few and long, and for those whose dQ fits into what
  // a second round of dK/dV leaves idle.
  // Two launches -> one, us: 16 / 4 heads, 777 tokens (168 workgroups) 83 -> 55; 24 heads, 1100 tokens (324) 92 -> 103, causal
  // 86 -> 61; 32 heads, 777 (336) 69 -> 80, causal 69 -> 48; causal 8 x 256 (384) 50 -> 52.5; wide 500 + 700 (320) 89 -> 78, 1300 (368)
  // 147 both; causal 1100 (288 of dK/dV, 432) 91 -> 82; 1500 (384, 576) 168 -> 170, causal 117 -> 121.
  const int both = p.kv_wgs + p.q_wgs;
  const int at_once = p.wide ? NUM_CU * 5 / 4 : a.causal && p.qtiles >= 3 * a.S ? NUM_CU * 3 / 2 : NUM_CU;
  p.together = !a.in_place && (same_wgs || both <= at_once || (p.kv_wgs > NUM_CU && both <= 2 * NUM_CU));
  if (!p.together && !same_wgs) p.q_wgs = p.qtiles * a.Hq;   // a kernel of its own, two workgroups per CU
  return p;
}

template <int DH>
bm_status bwd_launch(const AttnArgs& a, const void* o, const void* d_o, const float* lse, void* dq,
                     void* dk, void* dv, int ldd, float* delta, hipStream_t st) {
  const int ldo = a.Hq * a.dh;
  const int ldd_kv = a.ld_dkv ? a.ld_dkv : ldd;
  const float scale = 1.0f / sqrtf((float)a.dh);
  const float sl2 = scale * LOG2E;
  const long n = (long)a.T * a.Hq;
  if (n > 0)
    hipLaunchKernelGGL((fa_delta_kernel<DH>), dim3(cdiv(n * DeltaLanes<DH>::N, 256)), dim3(256), 0, st, (const bf16_t*)o,
                       (const bf16_t*)d_o, ldo, delta, a.T, a.Hq);
  const BwdPlan p = bwd_plan(a);
  const bool wide = p.wide, alt = p.alt;
  const int gsplit = p.gsplit;
  float* part = delta + align_up((size_t)a.Hq * a.T, 64);      // after the delta plane
  const int Tk = a.kv_T();
  // a key tile runs as long as its sequence has queries, a query tile as long as it has keys
  const SeqOrder ord_kv = make_seq_order(a.kv_cu_host(), a.cu_host, a.S, p.key_rows, !a.causal);
  const SeqOrder ord_q = make_seq_order(a.cu_host, a.kv_cu_host(), a.S, p.query_rows, !a.causal);
  // workgroups of dK/dV, then of dQ
  auto launch = [&](int kv, int q) {
    auto go = [&](auto kern, int threads) {
      hipLaunchKernelGGL(kern, dim3(kv + q), dim3(threads), 0, st, (const bf16_t*)a.q, (const bf16_t*)a.k, (const bf16_t*)a.v,
                         a.ld_qkv, a.kv_ld(), (const bf16_t*)d_o, ldo, lse, (const float*)delta, a.cu_dev, a.kv_cu_dev(), a.S,
                         (bf16_t*)dq, ldd, (bf16_t*)dk, (bf16_t*)dv, ldd_kv, a.T, Tk, a.Hkv, a.Hq / a.Hkv, scale, sl2, gsplit, part,
                         kv, ord_kv, ord_q);
    };
    if (kv + q == 0) return;
    if constexpr (DH <= 64) {
      go(a.causal ? fa_bwd_joint_kernel<DH, true> : fa_bwd_joint_kernel<DH, false>, 256);
    } else if constexpr (DH == 128) {
      if (wide && alt) go(a.causal ? fa_bwd_joint512_kernel<DH, true, true, true> : fa_bwd_joint512_kernel<DH, false, true, true>, 512);
      else if (wide) go(a.causal ? fa_bwd_joint512_kernel<DH, true, true, false> : fa_bwd_joint512_kernel<DH, false, true, false>, 512);
      else if (alt) go(a.causal ? fa_bwd_joint512_kernel<DH, true, false, true> : fa_bwd_joint512_kernel<DH, false, false, true>, 512);
      else go(a.causal ? fa_bwd_joint512_kernel<DH, true, false, false> : fa_bwd_joint512_kernel<DH, false, false, false>, 512);
    } else {
      go(a.causal ? fa_bwd_joint512_kernel<DH, true, false, false> : fa_bwd_joint512_kernel<DH, false, false, false>, 512);
    }
  };
  if (p.together) {
    launch(p.kv_wgs, p.q_wgs);
  } else {
    launch(p.kv_wgs, 0);
    bool same_wgs = true;
    if constexpr (DH > 64) same_wgs = alt;
    if (same_wgs) {
      launch(0, p.q_wgs);
    } else if constexpr (DH > 64) {
      if (p.q_wgs > 0) {
        auto kern = a.causal ? fa_bwd_dq_kernel<DH, true> : fa_bwd_dq_kernel<DH, false>;
        hipLaunchKernelGGL(kern, dim3(p.q_wgs), dim3(256), 0, st, (const bf16_t*)a.q, (const bf16_t*)a.k, (const bf16_t*)a.v,
                           a.ld_qkv, a.kv_ld(), (const bf16_t*)d_o, ldo, lse, (const float*)delta, a.cu_dev, a.kv_cu_dev(), a.S,
                           (bf16_t*)dq, ldd, a.T, a.Hq, a.Hq / a.Hkv, scale, sl2, ord_q);
      }
    }
  }
  if (gsplit > 1 && p.kv_wgs > 0) {
    const long n4 = (long)Tk * a.Hkv * a.dh / 4;
    hipLaunchKernelGGL(fa_dkdv_reduce_kernel, dim3(cdiv(n4, 256)), dim3(256), 0, st, part, gsplit, Tk,
                       a.Hkv * a.dh, (bf16_t*)dk, (bf16_t*)dv, ldd_kv);
  }
  BM_CHECK_LAUNCH("fa_bwd");
  return BM_OK;
}

}  // namespace

bool attention_mfma_supported(const AttnArgs& a) {
  return a.dtype == BM_DTYPE_BF16 && (a.dh == 64 || a.dh == 72 || a.dh == 128) && a.ld_qkv % 8 == 0 &&
         a.kv_ld() % 8 == 0;
}

bm_status attention_forward_mfma(const AttnArgs& a, void* o, float* lse, hipStream_t st) {
  if (a.dh == 128) return fwd_launch<128>(a, o, lse, st);
  if (a.dh == 72) return fwd_launch<72>(a, o, lse, st);
  return fwd_launch<64>(a, o, lse, st);
}

void attention_mfma_plan(const AttnArgs& a, int* fwd_rows, int* dq_rows, int* dkdv_rows) {
  const bool alt = a.dh != 72 && queries_alternating(a);
  *fwd_rows = alt ? AQ : FQ;
  *dq_rows = alt && a.dh == 128 ? AQ : FQ;
  *dkdv_rows = a.dh == 128 && dkdv_wide(a) ? WIDE_KEYS : BK_KEYS;
}

void attention_mfma_backward_plan(const AttnArgs& a, int* launches, int* dkdv_wgs, int* dq_wgs) {
  const BwdPlan p = bwd_plan(a);
  *launches = p.together ? 1 : 2;
  *dkdv_wgs = p.kv_wgs;
  *dq_wgs = p.q_wgs;
}

size_t attention_backward_mfma_scratch_bytes(int Hq, int Hkv, int dh, int Tq, int Tk) {
  // the delta plane of the query rows, then room for the fp32 dK/dV partials of the largest
  // q-head split
  const size_t delta = align_up((size_t)Hq * Tq, 64) * sizeof(float);
  const int group = Hq / Hkv;
  const size_t part = group > 1 ? (size_t)group * 2 * Tk * Hkv * dh * sizeof(float) : 0;
  return align_up(delta + part, 256);
}

bm_status attention_backward_mfma(const AttnArgs& a, const void* o, const void* d_o, const float* lse,
                                  void* dq, void* dk, void* dv, int ld_dqkv, void* scratch,
                                  size_t, hipStream_t st) {
  if (a.dh == 128) return bwd_launch<128>(a, o, d_o, lse, dq, dk, dv, ld_dqkv, (float*)scratch, st);
  if (a.dh == 72) return bwd_launch<72>(a, o, d_o, lse, dq, dk, dv, ld_dqkv, (float*)scratch, st);
  return bwd_launch<64>(a, o, d_o, lse, dq, dk, dv, ld_dqkv, (float*)scratch, st);
}

}  // namespace bm
