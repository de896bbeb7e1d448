// bf16 GEMM for large and medium tiles: two groups of wavefronts that take turns.
//
// A workgroup has eight wavefronts, two on every SIMD: group 0 (wavefronts 0-3) and group 1 (4-7).
// Work goes in phases with a workgroup barrier behind each; group 1 runs one phase behind group 0,
// so that in every phase one wavefront of a SIMD issues nothing but MFMAs (32 of them, 512 clocks)
// while the other one does everything else -- fragment reads for its next MFMAs, and the loads that
// bring later slices straight from memory into LDS.  No memory instruction ever stands in front of
// an MFMA of its own wavefront, and no wavefront holds staging registers.
//
// What this buys over one wavefront per SIMD that interleaves both (register-staged slices, four
// wavefronts of 128x128): NT 8192x12288x4096 1400 -> 1560 TFLOP/s, NN 8192x4096x12288 1390 -> 1560,
// TN 12288x4096x8192 1230 -> 1370, NT 16384x3072x1024 1150 -> 1280 (random operands, one box).  It is
// bound by the power the matrix pipe draws: priorities, the order of a phase's memory instructions
// and the tile order changed nothing.
//
// Loads that write LDS: lane l of a wavefront fills bytes 16 l .. 16 l + 15 of a 1 KiB run, so the
// swizzle sits on the global side: the lane that owns a slot fetches the chunk that belongs there.
// They are asm statements, invisible to the compiler's wait-count bookkeeping, which would make every
// fragment read wait for all of them; the waits stand in the phases instead, and since the loads of
// a wavefront return in order a wait for "at most n outstanding" names the ones that must have landed.
#include "gemm_tile.h"

#include <atomic>

namespace bm {

namespace {

constexpr int THREADS = 512;

template <int N> using Int = std::integral_constant<int, N>;

template <int N> __device__ inline void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }
__device__ inline void wait_fragments() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
__device__ inline void end_phase() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}
__device__ inline void load_to_lds(const bf16_t* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(off), "s"(base) : "memory", "m0");
}

// the source of a row, or that of the first row where there is none (the rows that fill up a group)
__device__ inline int source_row(const int32_t* source, int row, int src_rows) {
  const int s = source[row];
  return (uint32_t)s < (uint32_t)src_rows ? s : min(max(source[0], 0), src_rows - 1);
}

// LDS layouts of a region of R rows x 64 k (the swizzles keep fragment reads free of bank conflicts):
//   k-contiguous operand  [row][64 k]: 16-byte chunk c of row r sits at c ^ ((r >> 1) & 7)
//   transposed operand    [k][R rows]: chunk c of k-row k sits at c ^ ((k & 3) << 2) ^ (((k >> 3) & 1) << 1)
// A region is filled in R/64 loads per wavefront; load i of wavefront w writes the 1 KiB run i*8 + w.
template <int R, bool TR>
struct Region {
  static constexpr int LOADS = R / 64;
  static constexpr uint32_t BYTES = R * BK * 2;
  static constexpr int CPR = TR ? R / 8 : KCH;           // chunks per LDS row
  static constexpr int RPL = 64 / CPR;                   // LDS rows per load
  uint32_t off[LOADS];                                   // byte offset from the slice's base pointer
  // LDS row and global chunk of this lane in load i
  static __device__ inline void place(int i, int wave, int lane, int* row, int* chunk) {
    const int r = (i * 8 + wave) * RPL + lane / CPR;
    *row = r;
    *chunk = (lane % CPR) ^ (TR ? ((r & 3) << 2) ^ (((r >> 3) & 1) << 1) : (r >> 1) & 7);
  }
  // row0: this region's first row in the tile; rows past rows_left (counted from the tile's first row)
  // are clamped into the matrix: their products are never stored.
  // half > 0 (k-contiguous only): rows are gathered from two ranges F rows apart -- within every run of
  // 2*half tile rows the first half come from f0.. and the second from F + f0.. (gate and up rows of a
  // SwiGLU weight); offsets are then relative to the matrix's first row.
  // source (k-contiguous only): where the tile's rows lie in a matrix of src_rows rows; offsets are then relative to its first row
  __device__ inline void init(int ld, int row0, int rows_left, int wave, int lane, int half = 0, int F = 0, int f0 = 0,
                              const int32_t* source = nullptr, int src_rows = 0) {
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
      int r, c;
      place(i, wave, lane, &r, &c);
      if (TR) {
        int row = row0 + c * 8;
        if (row >= rows_left) row = 0;
        off[i] = ((uint32_t)r * (uint32_t)ld + (uint32_t)row) * 2u;
      } else {
        int row = min(row0 + r, rows_left - 1);
        if (half > 0) row = (r / half & 1) * F + f0 + (r / (2 * half)) * half + r % half;
        if (source) row = source_row(source, row, src_rows);
        off[i] = ((uint32_t)row * (uint32_t)ld + (uint32_t)c * 8u) * 2u;
      }
    }
  }
  // k_left < 64: a slice that ends inside the k range; what lies past it is fetched from its last
  // valid k (row or chunk) and zeroed in the fragments
  template <bool CUT, int FIRST = 0, int COUNT = LOADS>
  __device__ inline void load(const bf16_t* base, int ld, int k_left, uint32_t lds, int wave, int lane) const {
#pragma unroll
    for (int i = FIRST; i < FIRST + COUNT; ++i) {
      uint32_t o = off[i];
      if (CUT && k_left < BK) {
        int r, c;
        place(i, wave, lane, &r, &c);
        if (TR) { if (r >= k_left) o -= (uint32_t)(r - (k_left - 1)) * (uint32_t)ld * 2u; }
        else if (c * 8 >= k_left) o -= (uint32_t)(c * 8 - (k_left - 8)) * 2u;
      }
      load_to_lds(base, o, lds + (i * 8 + wave) * 1024);
    }
  }
};

// The same for a transposed operand whose k rows are read from their source rows: those of the tile's k range lie in LDS, and
// the ones of a load are fetched a phase ahead of it.
template <int R, int FIRST, int COUNT>
struct SourceLoads {
  using Reg = Region<R, true>;
  int row[COUNT];
  __device__ inline void fetch(const int32_t* rows, int j, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < COUNT; ++i) row[i] = rows[j * BK + ((FIRST + i) * 8 + wave) * Reg::RPL + lane / Reg::CPR];
  }
  // col: byte offset of this lane's chunk in a row, the same in every load
  __device__ inline void load(const bf16_t* base, uint32_t row_bytes, uint32_t col, uint32_t lds, int wave) const {
#pragma unroll
    for (int i = 0; i < COUNT; ++i) load_to_lds(base, (uint32_t)row[i] * row_bytes + col, lds + ((FIRST + i) * 8 + wave) * 1024);
  }
};

// 16(row) x 32(k) fragments of v_mfma_f32_16x16x32_bf16 from a region of R rows: lane l holds row l%16
// and k = (l/16)*8 .. +7.  NB blocks of 16 rows from row0 on; block q, k-step ks.
template <int R, bool TR, int NB>
struct Fragments {
  static constexpr int NA = TR ? NB : 2;
  uint32_t addr[NA];
  __device__ inline void init(int row0, int lane) {
    const int gi = lane >> 4, s = lane & 15;
#pragma unroll
    for (int q = 0; q < NA; ++q) {
      if (TR) {
        // the 16 lanes of group gi read a 4(k) x 16(row) block, 8 bytes each; the transpose read
        // hands lane s row s with 4 consecutive k; two reads give 8 k
        const int k = gi * 8 + (s >> 2);
        const int c = (row0 / 8 + q * 2 + ((s & 3) >> 1)) ^ ((s >> 2) << 2) ^ ((gi & 1) << 1);
        addr[q] = k * (R * 2) + c * 16 + (s & 1) * 8;
      } else {
        addr[q] = (row0 + s) * (BK * 2) + ((q * 4 + gi) ^ (s >> 1)) * 16;
      }
    }
  }
  __device__ inline bf16x8 read(const unsigned char* smem, int q, int ks, uint32_t base) const {
    if (TR) {
      const unsigned char* p = smem + addr[q] + base + ks * (32 * R * 2);
      s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)p);
      s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 4 * R * 2));
      union { struct { s16x4 a, b; } s; bf16x8 v; } u;
      u.s.a = lo; u.s.b = hi;
      return u.v;
    }
    return *reinterpret_cast<const bf16x8*>(smem + addr[ks] + base + q * (16 * BK * 2));
  }
};

// What lies past the k range of a cut slice is zeroed in the fragments: a mask over the 8 k of this lane in k-step
// ks, one AND per register.  A compare and a select per element were a thousand instructions that a tile fetches and
// issues for its last slice alone: 4096x4096, K = 72, NT 16.5 -> 11.5 us (K = 64: 10.2), K = 400 24.3 -> 21.2;
// TN 22016x4096 over 777 rows 271 -> 244.
__device__ inline u32x4 cut_mask(int ks, int k_left, int lane) {
  const int left = k_left - ks * 32 - (lane >> 4) * 8;
  u32x4 m;
#pragma unroll
  for (int e = 0; e < 4; ++e) m[e] = left > 2 * e + 1 ? 0xffffffffu : left > 2 * e ? 0xffffu : 0u;
  return m;
}
__device__ inline void cut_fragment(bf16x8& f, const u32x4& mask) {
  union { bf16x8 f; u32x4 u; } x{f};
  x.u &= mask;
  f = x.f;
}

// Accumulators start as the product of zero operands: written by ordinary instructions they would need
// wait states in front of the first MFMA that the compiler, which does not know the asm statements
// are MFMAs, would not leave.
template <int FM, int FN>
__device__ inline void clear(f32x4 (&acc)[FM][FN]) {
  bf16x8 z = {};
  asm volatile("s_nop 7" : "+v"(z));
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) mfma16_first(acc[i][j], z, z);
}

// ---- 256x256 tile of NT and NN.  Each wavefront owns 128x64: 64 rows in each half of A, 64 columns of B.  A slice is
// two phases per group (first and second half of A); LDS holds two slices, and a slice's first half
// of A with B, and its second half, are re-filled as soon as both groups have read them: loads are
// in flight for more than a slice (4 to 5 phases of 512 clocks).
template <bool B_TR, int EPI, bool CUT, bool SOURCE = false>
__device__ __forceinline__ void alt256_tile(const GemmParams& p, const TileJob& job) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RegA = Region<128, false>;
  using RegB = Region<256, B_TR>;
  constexpr uint32_t A1 = RegA::BYTES, B0 = 2 * RegA::BYTES, BUF = B0 + RegB::BYTES;
  constexpr int LATE = RegA::LOADS, EARLY = RegA::LOADS + RegB::LOADS;      // loads of a slice's two parts
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;                                   // wm is the group
  if (job.kbeg >= job.kend) return;
  const int m0 = job.m0, n0 = job.n0, n = (job.kend - job.kbeg + BK - 1) / BK;
  const int k_left = job.kend - job.kbeg - (n - 1) * BK;                     // of the last slice
  constexpr bool SWF = EPI == EPI_SWIGLU_FWD;

  RegA ra0, ra1;
  RegB rb;
  const int32_t* source = SOURCE && p.source ? p.source + m0 : nullptr;
  ra0.init(p.lda, 0, p.M - m0, wave, lane, 0, 0, 0, source, p.src_rows);
  ra1.init(p.lda, 128, p.M - m0, wave, lane, 0, 0, 0, source, p.src_rows);
  if (SWF) rb.init(p.ldb, 0, 256, wave, lane, 32, p.N / 2, job.tn * 128);
  else rb.init(p.ldb, 0, p.N - n0, wave, lane);
  const bf16_t* a_base = job.A + (source ? (size_t)0 : (size_t)m0 * p.lda) + job.kbeg;
  const bf16_t* b_base = B_TR ? job.B + (size_t)job.kbeg * p.ldb + n0
                              : job.B + (SWF ? (size_t)0 : (size_t)n0 * p.ldb) + job.kbeg;
  const size_t a_step = BK, b_step = B_TR ? (size_t)BK * p.ldb : (size_t)BK;
  auto load_early = [&](int j, uint32_t buf) {
    const int left = CUT && j == n - 1 ? k_left : BK;
    rb.template load<CUT>(b_base + (size_t)j * b_step, p.ldb, left, buf + B0, wave, lane);
    ra0.template load<CUT>(a_base + (size_t)j * a_step, p.lda, left, buf, wave, lane);
  };
  auto load_late = [&](int j, uint32_t buf) {
    ra1.template load<CUT>(a_base + (size_t)j * a_step, p.lda, CUT && j == n - 1 ? k_left : BK, buf + A1, wave, lane);
  };

  Fragments<128, false, 4> fa;
  Fragments<256, B_TR, 4> fb;
  fa.init(wm * 64, lane);
  fb.init(wn * 64, lane);
  bf16x8 af[2][4], bf[2][4];
  f32x4 acc[8][4];
  auto multiply = [&](auto half_t) {
    constexpr int H = decltype(half_t)::value * 4;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) mfma16(acc[H + i][j], bf[ks][j], af[ks][i]);
  };
  // COME: slices that follow this one (2: two or more, 0: this is the last)
  auto slice = [&](auto come_t, int j) {
    constexpr int COME = decltype(come_t)::value;
    const uint32_t buf = (j & 1) * BUF;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int q = 0; q < 4; ++q) bf[ks][q] = fb.read(smem, q, ks, buf + B0);
#pragma unroll
      for (int q = 0; q < 4; ++q) af[ks][q] = fa.read(smem, q, ks, buf);
    }
    if (COME >= 1) load_late(j + 1, buf ^ BUF);
    wait_fragments();
    if (CUT && COME == 0 && k_left < BK) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const u32x4 mask = cut_mask(ks, k_left, lane);
#pragma unroll
        for (int q = 0; q < 4; ++q) { cut_fragment(bf[ks][q], mask); cut_fragment(af[ks][q], mask); }
      }
    }
    // the second half of A of this slice is read next: everything older than the loads requested
    // since (the next slice's two parts) must have landed
    wait_loads<COME >= 1 ? EARLY + LATE : 0>();
    end_phase();
    multiply(Int<0>{});
    wait_loads<COME >= 1 ? EARLY + LATE : 0>();
    end_phase();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int q = 0; q < 4; ++q) af[ks][q] = fa.read(smem, q, ks, buf + A1);
    if (COME >= 2) load_early(j + 2, buf);
    wait_fragments();
    if (CUT && COME == 0 && k_left < BK) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const u32x4 mask = cut_mask(ks, k_left, lane);
#pragma unroll
        for (int q = 0; q < 4; ++q) cut_fragment(af[ks][q], mask);
      }
    }
    if (COME == 0) { end_phase(); return; }                 // the last MFMAs belong to the epilogue
    // next: the following slice's first half of A and B
    wait_loads<COME >= 2 ? EARLY + LATE : LATE>();
    end_phase();
    multiply(Int<1>{});
    wait_loads<COME >= 2 ? EARLY + LATE : LATE>();
    end_phase();
  };
  load_early(0, 0);
  load_late(0, 0);
  if (n > 1) load_early(1, BUF);
  clear(acc);                                               // under the latency of the first loads
  if (n > 1) wait_loads<EARLY + LATE>();
  else wait_loads<0>();
  end_phase();
  if (wm == 1) end_phase();                                 // group 1 stays one phase behind
  const bool full = m0 + 256 <= p.M && n0 + 256 <= p.N;
  for (int j = 0; j < n - 2; ++j) slice(Int<2>{}, j);
  if (n > 1) slice(Int<1>{}, n - 2);
  slice(Int<0>{}, n - 1);
  gemm_epilogue<EPI, 8, 4>(p, acc, reinterpret_cast<float*>(smem) + wave * epilogue_stage_floats<4>(), lane,
                           n0 + wn * 64, job.tn * 128 + wn * 32, job.split, job.c_off, full,
                           [&](int i) { return m0 + (i >> 2) * 128 + wm * 64 + (i & 3) * 16; },
                           [&] {
                             multiply(Int<1>{});
                             // group 0 writes its strips over the buffers group 1 has just read
                             if (wm == 0) end_phase();
                           });
}

// ---- 256x256 tile of a weight gradient (TN).  Both operands lie [k][row] in LDS, so a slice is cut along k: each of
// its two phases per group reads 12 fragments of 32 k (8 of A, 4 of B) and multiplies 8x4 blocks.  Cut along
// the rows of A as above, the phases read 16 and 8 fragments, and 32 transpose reads with their latency do not fit under
// 512 clocks of MFMAs.  A slice of a tile that has the chip to itself: 1.17 us cut along the rows, 0.96 along k (NT 0.87);
// with all CUs at work 1.45 and 1.33 (power).  12288x4096 over 8192 rows 621 -> 604 us, 22016x4096 over 777 247 -> 241.
// The first 32 k of a slice are re-filled while its last 32 are read, and the other way round.  (K-contiguous operands
// are cut along the rows because half a slice of theirs would be half of every 128-byte line.)
// SOURCE: 1 or 2 where the k rows of A or B are read from their source rows (whole slices only).  The table of source rows costs a tile
// about a microsecond in front of its first loads and four LDS reads a slice; a sorted copy costs its own pass and 268 MB to
// be read back (65536 rows of 2048): up 1536x2048 with the pass 870 -> 755 us, down 2048x768 500 -> 405.
// The contraction ends at the last routed row: the rows that fill up a group read a row of a token, and an infinity of that token
// would meet their zeros as a NaN (8192 tokens, 128 experts: 4268 us a pass with those rows masked in whole blocks, 4231 without them).
template <int EPI, bool CUT, int SOURCE = 0>
__device__ __forceinline__ void alt256_tn_tile(const GemmParams& p, const TileJob& job) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using Reg = Region<256, true>;
  constexpr uint32_t B0 = Reg::BYTES, BUF = 2 * Reg::BYTES;
  constexpr int HL = Reg::LOADS;                                             // loads of half a slice, A and B
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;                                   // wm is the group
  if (job.kbeg >= job.kend) return;
  const int m0 = job.m0, n0 = job.n0;
  int n = (job.kend - job.kbeg + BK - 1) / BK;
  int k_left = job.kend - job.kbeg - (n - 1) * BK;                           // of the last slice

  Reg ra, rb;
  ra.init(p.lda, 0, p.M - m0, wave, lane);
  rb.init(p.ldb, 0, p.N - n0, wave, lane);
  const bf16_t* a_base = job.A + (size_t)job.kbeg * p.lda + m0;
  const bf16_t* b_base = job.B + (size_t)job.kbeg * p.ldb + n0;
  const size_t a_step = (size_t)BK * p.lda, b_step = (size_t)BK * p.ldb;
  // source rows of the tile's k range in LDS behind the slices, and those of the next loads of either half of a slice
  int32_t* rows = reinterpret_cast<int32_t*>(smem + 2 * BUF);
  SourceLoads<256, 0, HL / 2> next0;
  SourceLoads<256, HL / 2, HL / 2> next1;
  const uint32_t src_bytes = (uint32_t)(SOURCE == 1 ? p.lda : p.ldb) * 2u;
  uint32_t src_col = 0;
  if (SOURCE) {
    int r, c;
    Reg::place(0, wave, lane, &r, &c);
    const int first = SOURCE == 1 ? m0 : n0, left = (SOURCE == 1 ? p.M : p.N) - first;
    src_col = (uint32_t)(c * 8 < left ? c * 8 : 0) * 2u;
  }
  const bf16_t* src_base = SOURCE == 1 ? job.A + m0 : job.B + n0;
  auto load_b = [&](auto half_t, int j, uint32_t buf) {
    constexpr int FIRST = decltype(half_t)::value * (HL / 2);
    const int left = CUT && j == n - 1 ? k_left : BK;
    rb.template load<CUT, FIRST, HL / 2>(b_base + (size_t)j * b_step, p.ldb, left, buf + B0, wave, lane);
  };
  auto load_a = [&](auto half_t, int j, uint32_t buf) {
    constexpr int FIRST = decltype(half_t)::value * (HL / 2);
    const int left = CUT && j == n - 1 ? k_left : BK;
    ra.template load<CUT, FIRST, HL / 2>(a_base + (size_t)j * a_step, p.lda, left, buf, wave, lane);
  };
  auto load_source = [&](auto half_t, uint32_t buf) {
    const uint32_t at = buf + (SOURCE == 1 ? 0 : B0);
    if constexpr (decltype(half_t)::value == 0) next0.load(src_base, src_bytes, src_col, at, wave);
    else next1.load(src_base, src_bytes, src_col, at, wave);
  };
  auto fetch_rows = [&](auto half_t, int j) {
    if constexpr (SOURCE != 0) {
      if constexpr (decltype(half_t)::value == 0) next0.fetch(rows, j, wave, lane);
      else next1.fetch(rows, j, wave, lane);
    }
  };
  auto load_half = [&](auto half_t, int j, uint32_t buf) {
    if constexpr (SOURCE == 2) load_source(half_t, buf); else load_b(half_t, j, buf);
    if constexpr (SOURCE == 1) load_source(half_t, buf); else load_a(half_t, j, buf);
  };

  // rows wm*64.. of each half of A: the second half lies 128 rows on in every k row
  Fragments<256, true, 4> fa, fb;
  fa.init(wm * 64, lane);
  fb.init(wn * 64, lane);
  bf16x8 af[8], bf[4];
  f32x4 acc[8][4];
  auto multiply = [&] {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) mfma16(acc[i][j], bf[j], af[i]);
  };
  auto read = [&](auto ks_t, uint32_t buf) {
    constexpr int KS = decltype(ks_t)::value;
#pragma unroll
    for (int q = 0; q < 4; ++q) bf[q] = fb.read(smem, q, KS, buf + B0);
#pragma unroll
    for (int q = 0; q < 4; ++q) af[q] = fa.read(smem, q, KS, buf);
#pragma unroll
    for (int q = 0; q < 4; ++q) af[4 + q] = fa.read(smem, q, KS, buf + 128 * 2);
  };
  auto cut = [&](int ks) {
    const u32x4 mask = cut_mask(ks, k_left, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) cut_fragment(bf[q], mask);
#pragma unroll
    for (int q = 0; q < 8; ++q) cut_fragment(af[q], mask);
  };
  // COME: slices that follow this one (2: two or more, 0: this is the last).  A wait names the half slice that is read
  // next: everything older than the two halves requested since must have landed.
  auto slice = [&](auto come_t, int j) {
    constexpr int COME = decltype(come_t)::value;
    const uint32_t buf = (j & 1) * BUF;
    read(Int<0>{}, buf);
    if (COME >= 1) load_half(Int<1>{}, j + 1, buf ^ BUF);
    if (COME >= 2) fetch_rows(Int<0>{}, j + 2);
    wait_fragments();
    if ((CUT || SOURCE) && COME == 0 && k_left < BK) cut(0);
    wait_loads<COME >= 1 ? 2 * HL : 0>();
    end_phase();
    multiply();
    wait_loads<COME >= 1 ? 2 * HL : 0>();
    end_phase();
    read(Int<1>{}, buf);
    if (COME >= 2) { load_half(Int<0>{}, j + 2, buf); fetch_rows(Int<1>{}, j + 2); }
    wait_fragments();
    if ((CUT || SOURCE) && COME == 0 && k_left < BK) cut(1);
    if (COME == 0) { end_phase(); return; }                 // the last MFMAs belong to the epilogue
    wait_loads<COME >= 2 ? 2 * HL : HL>();
    end_phase();
    multiply();
    wait_loads<COME >= 2 ? 2 * HL : HL>();
    end_phase();
  };
  if constexpr (SOURCE != 0) {
    // the other operand's first slice is on its way while the table is filled
    if constexpr (SOURCE == 2) { load_a(Int<0>{}, 0, 0); load_a(Int<1>{}, 0, 0); }
    else { load_b(Int<0>{}, 0, 0); load_b(Int<1>{}, 0, 0); }
    for (int i = threadIdx.x; i < n * BK; i += THREADS) rows[i] = source_row(p.source + job.kbeg, i, p.src_rows);
    int routed = n * BK - MOE_PAD;
#pragma unroll
    for (int i = 0; i < MOE_PAD; i += WAVE)
      routed += __popcll(__ballot((uint32_t)p.source[job.kend - MOE_PAD + i + lane] < (uint32_t)p.src_rows));
    routed = __builtin_amdgcn_readfirstlane(max(routed, 1));
    n = (routed + BK - 1) / BK;
    k_left = routed - (n - 1) * BK;
    __syncthreads();
    fetch_rows(Int<0>{}, 0);
    fetch_rows(Int<1>{}, 0);
    load_source(Int<0>{}, 0);
    load_source(Int<1>{}, 0);
    if (n > 1) {
      fetch_rows(Int<0>{}, 1);
      load_half(Int<0>{}, 1, BUF);
      fetch_rows(Int<1>{}, 1);
    }
    clear(acc);
    if (n > 1) wait_loads<HL + HL / 2>();
    else wait_loads<0>();
  } else {
    load_half(Int<0>{}, 0, 0);
    load_half(Int<1>{}, 0, 0);
    if (n > 1) load_half(Int<0>{}, 1, BUF);
    clear(acc);                                             // under the latency of the first loads
    if (n > 1) wait_loads<2 * HL>();
    else wait_loads<0>();
  }
  end_phase();
  if (wm == 1) end_phase();                                 // group 1 stays one phase behind
  const bool full = m0 + 256 <= p.M && n0 + 256 <= p.N;
  for (int j = 0; j < n - 2; ++j) slice(Int<2>{}, j);
  if (n > 1) slice(Int<1>{}, n - 2);
  slice(Int<0>{}, n - 1);
  gemm_epilogue<EPI, 8, 4>(p, acc, reinterpret_cast<float*>(smem) + wave * epilogue_stage_floats<4>(), lane,
                           n0 + wn * 64, 0, job.split, job.c_off, full,
                           [&](int i) { return m0 + (i >> 2) * 128 + wm * 64 + (i & 3) * 16; },
                           [&] {
                             multiply();
                             // group 0 writes its strips over the buffers group 1 has just read
                             if (wm == 0) end_phase();
                           });
}

template <int EPI, bool CUT>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt256_tn_kernel(GemmParams p) {
  alt256_tn_tile<EPI, CUT>(p, locate_tile<256, 256>(p, blockIdx.x));
}

// Grouped weight gradients with one operand read from its source rows.
template <int SOURCE>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt256_tn_source_kernel(GemmParams p) {
  TileJob job = locate_tile<256, 256>(p, blockIdx.x);
  job.kend = min(job.kend, job.kbeg + MOE_SOURCE_ROWS);       // (no group of that many source rows is longer)
  alt256_tn_tile<EPI_ADD, false, SOURCE>(p, job);
}

// Several weight gradients in one grid.
template <bool CUT>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt256_tn_parts_kernel(TnParts g) {
  // One round of tiles with one k range lies in one list, of which every XCD takes a run: an XCD that took a run of every
  // part would fetch twice the panels (a block of 1024 columns, 5477 rows: 161 -> 146 us).  Over several rounds a
  // run of every part is better: then all XCDs walk the same operands at a time (the stage of four microbatches
  // 155.2 -> 154.7 ms).
  const int pid = blockIdx.x, id = pid < g.one_list ? xcd_run(pid, g.one_list) : pid;
  int i = 0;
  while (i + 1 < g.n && id >= g.part[i + 1].first_wg) ++i;
  const TnParts::Part& q = g.part[i];
  GemmParams p{};
  p.A = q.A; p.B = q.B; p.C = q.C; p.partial = q.partial;
  p.M = q.M; p.N = q.N; p.K = q.K; p.lda = q.lda; p.ldb = q.ldb; p.ldc = q.ldc;
  p.tiles_m = q.tiles_m; p.tiles_n = q.tiles_n; p.splits = q.splits; p.k_per_split = q.k_per_split;
  p.xcd_split = q.xcd_split;
  if (p.splits > 1) {
    alt256_tn_tile<EPI_PARTIAL, CUT>(p, locate_tile<256, 256>(p, id - q.first_wg));
  } else {
    int tm, tn, t = id - q.first_wg;
    if (g.one_list == 0) t = xcd_run(t, q.tiles_m * q.tiles_n);
    grouped_tile<4>(t, q.tiles_m, q.tiles_n, &tm, &tn);
    alt256_tn_tile<EPI_ADD, CUT>(p, tile_job<256, 256>(p, 0, tm, tn));
  }
}

// ---- 128x256 and 256x128 tiles: each wavefront owns 64x64 and a slice is one phase per group.  LDS holds
// three slices; the loads of slice j+2 go out while slice j is read.
template <int BM, int BN, bool A_TR, bool B_TR, int EPI, bool CUT, bool SOURCE = false>
__device__ __forceinline__ void alt128_tile(const GemmParams& p, const TileJob& job) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  using RegA = Region<BM, A_TR>;
  using RegB = Region<BN, B_TR>;
  constexpr uint32_t B0 = RegA::BYTES, BUF = B0 + RegB::BYTES;
  constexpr int LOADS = RegA::LOADS + RegB::LOADS;
  constexpr int WN = BN / 64;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN, group = wave >> 2;
  if (job.kbeg >= job.kend) return;
  const int m0 = job.m0, n0 = job.n0, n = (job.kend - job.kbeg + BK - 1) / BK;
  const int k_left = job.kend - job.kbeg - (n - 1) * BK;
  constexpr bool SWF = EPI == EPI_SWIGLU_FWD;

  RegA ra;
  RegB rb;
  const int32_t* source = SOURCE && p.source ? p.source + m0 : nullptr;
  ra.init(p.lda, 0, p.M - m0, wave, lane, 0, 0, 0, source, p.src_rows);
  if (SWF) rb.init(p.ldb, 0, BN, wave, lane, 32, p.N / 2, job.tn * (BN / 2));
  else rb.init(p.ldb, 0, p.N - n0, wave, lane);
  const bf16_t* a_base = A_TR ? job.A + (size_t)job.kbeg * p.lda + m0
                              : job.A + (source ? (size_t)0 : (size_t)m0 * p.lda) + job.kbeg;
  const bf16_t* b_base = B_TR ? job.B + (size_t)job.kbeg * p.ldb + n0
                              : job.B + (SWF ? (size_t)0 : (size_t)n0 * p.ldb) + job.kbeg;
  const size_t a_step = A_TR ? (size_t)BK * p.lda : (size_t)BK, b_step = B_TR ? (size_t)BK * p.ldb : (size_t)BK;
  auto load = [&](int j, uint32_t buf) {
    const int left = CUT && j == n - 1 ? k_left : BK;
    rb.template load<CUT>(b_base + (size_t)j * b_step, p.ldb, left, buf + B0, wave, lane);
    ra.template load<CUT>(a_base + (size_t)j * a_step, p.lda, left, buf, wave, lane);
  };

  Fragments<BM, A_TR, 4> fa;
  Fragments<BN, B_TR, 4> fb;
  fa.init(wm * 64, lane);
  fb.init(wn * 64, lane);
  bf16x8 af[2][4], bf[2][4];
  f32x4 acc[4][4];
  auto multiply = [&] {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) mfma16(acc[i][j], bf[ks][j], af[ks][i]);
  };
  uint32_t cur = 0;                                          // buffer of the slice to be read next
  auto next_buf = [&](uint32_t b) { return b == 2 * BUF ? 0u : b + BUF; };
  auto slice = [&](auto come_t, int j) {
    constexpr int COME = decltype(come_t)::value;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int q = 0; q < 4; ++q) bf[ks][q] = fb.read(smem, q, ks, cur + B0);
#pragma unroll
      for (int q = 0; q < 4; ++q) af[ks][q] = fa.read(smem, q, ks, cur);
    }
    const uint32_t nxt = next_buf(cur);
    if (COME >= 2) load(j + 2, next_buf(nxt));
    wait_fragments();
    if (CUT && COME == 0 && k_left < BK) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const u32x4 mask = cut_mask(ks, k_left, lane);
#pragma unroll
        for (int q = 0; q < 4; ++q) { cut_fragment(bf[ks][q], mask); cut_fragment(af[ks][q], mask); }
      }
    }
    cur = nxt;
    if (COME == 0) { end_phase(); return; }                  // the last MFMAs belong to the epilogue
    wait_loads<COME >= 2 ? LOADS : 0>();                     // the next slice has landed
    end_phase();
    multiply();
    wait_loads<COME >= 2 ? LOADS : 0>();
    end_phase();
  };
  load(0, 0);
  if (n > 1) load(1, BUF);
  clear(acc);
  if (n > 1) wait_loads<LOADS>();
  else wait_loads<0>();
  end_phase();
  if (group == 1) end_phase();
  const bool full = m0 + BM <= p.M && n0 + BN <= p.N;
  for (int j = 0; j < n - 2; ++j) slice(Int<2>{}, j);
  if (n > 1) slice(Int<1>{}, n - 2);
  slice(Int<0>{}, n - 1);
  gemm_epilogue<EPI, 4, 4>(p, acc, reinterpret_cast<float*>(smem) + wave * epilogue_stage_floats<4>(), lane,
                           n0 + wn * 64, job.tn * (BN / 2) + wn * 32, job.split, job.c_off, full,
                           [&](int i) { return m0 + wm * 64 + i * 16; },
                           [&] {
                             multiply();
                             if (group == 0) end_phase();
                           });
}

template <bool B_TR, int EPI, bool CUT>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt256_kernel(GemmParams p) {
  alt256_tile<B_TR, EPI, CUT>(p, locate_tile<256, 256>(p, blockIdx.x));
}

template <int BM, int BN, bool A_TR, bool B_TR, int EPI, bool CUT>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt128_kernel(GemmParams p) {
  alt128_tile<BM, BN, A_TR, B_TR, EPI, CUT>(p, locate_tile<BM, BN>(p, blockIdx.x));
}

// Rows on tiles of two heights: the 256x256 tiles that fill whole rounds, and the rows that are left on 128x256, which end a
// round earlier than another one of 256x256 would (see mixed_rows()).
template <bool B_TR, int EPI, bool CUT>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt_mixed_kernel(GemmParams p) {
  const int big = p.big_rows * p.tiles_n;
  int tm, tn;
  if ((int)blockIdx.x < big) {
    tile_of_block(blockIdx.x, big, p.big_rows, p.tiles_n, &tm, &tn);
    alt256_tile<B_TR, EPI, CUT>(p, tile_job<256, 256>(p, 0, tm, tn));
  } else {
    const int rows = p.tiles_m - p.big_rows;
    tile_of_block((int)blockIdx.x - big, rows * p.tiles_n, rows, p.tiles_n, &tm, &tn);
    alt128_tile<128, 256, false, B_TR, EPI, CUT>(p, tile_job<128, 256>(p, 0, 2 * p.big_rows + tm, tn));
  }
}

// Grouped NT and NN (experts): two row blocks of a group share a 256x256 tile, the last one of an odd number takes 128x256.  How many
// tiles there are is known on the device only; the XCDs share those, not the capacity, whose end is empty (a tenth of
// it with 128 experts of 512 rows, all in the last XCD's run).  8192 tokens, 8 of 128 experts, against one 128x256 tile per row
// block: up 1536x2048 with SwiGLU 575 -> 460 us, its input gradient 565 -> 440, down 2048x768 330 -> 255, its input gradient with
// SwiGLU 350 -> 305; the outputs are the same bit for bit.  Bound by HBM (1.4 GB of weights and rows, 290 us) next to the MFMAs (300).
template <bool B_TR, int EPI, bool CUT>
__global__ __launch_bounds__(THREADS, 2) void gemm_alt_groups_kernel(GemmParams p) {
  const int row_tiles = p.row_tiles[0], total = row_tiles * p.tiles_n;
  if ((int)blockIdx.x >= total) return;
  int tm, tn;
  const int id = xcd_run(blockIdx.x, total);
  if (p.walk_rows == 2) grouped_tile<2>(id, row_tiles, p.tiles_n, &tm, &tn);
  else grouped_tile<4>(id, row_tiles, p.tiles_n, &tm, &tn);
  const int tile = p.row_tiles[1 + tm], block = tile >> 1;
  TileJob job;
  job.A = p.A; job.B = p.B + (long)p.tile_group[block] * p.b_group_stride;
  job.m0 = block * MOE_PAD; job.n0 = tn * 256; job.tn = tn;
  job.kbeg = 0; job.kend = p.K; job.split = 0; job.c_off = 0;
  p.M = job.m0 + (tile & 1 ? 2 : 1) * MOE_PAD;
  constexpr bool SOURCE = EPI == EPI_SWIGLU_FWD || EPI == EPI_SWIGLU_BWD;
  if (tile & 1) alt256_tile<B_TR, EPI, CUT, SOURCE>(p, job);
  else alt128_tile<MOE_PAD, 256, false, B_TR, EPI, CUT, SOURCE>(p, job);
}

template <int BM, int BN, bool A_TR, bool B_TR, int EPI, bool CUT>
bm_status launch_one(const GemmParams& p, hipStream_t st) {
  constexpr bool LARGE = BM == 256 && BN == 256;
  constexpr size_t lds = (size_t)(LARGE ? 2 : 3) * (BM + BN) * BK * sizeof(bf16_t);
  void (*kern)(GemmParams);
  if constexpr (LARGE && A_TR) kern = gemm_alt256_tn_kernel<EPI, CUT>;
  else if constexpr (LARGE) kern = gemm_alt256_kernel<B_TR, EPI, CUT>;
  else kern = gemm_alt128_kernel<BM, BN, A_TR, B_TR, EPI, CUT>;
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_relaxed)) {
    BM_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_done.store(true, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n * p.splits * p.grid_groups), dim3(THREADS), lds, st, p);
  BM_CHECK_LAUNCH("gemm_alt");
  return BM_OK;
}

// kernels that hold both a 256x256 and a 128x256 tile
template <bool GROUPS, bool B_TR, int EPI, bool CUT>
bm_status launch_two_heights(const GemmParams& p, hipStream_t st) {
  constexpr size_t lds = (size_t)3 * (128 + 256) * BK * sizeof(bf16_t);
  void (*kern)(GemmParams);
  if constexpr (GROUPS) kern = gemm_alt_groups_kernel<B_TR, EPI, CUT>;
  else kern = gemm_alt_mixed_kernel<B_TR, EPI, CUT>;
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_relaxed)) {
    BM_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_done.store(true, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n), dim3(THREADS), lds, st, p);
  BM_CHECK_LAUNCH("gemm_alt_two_heights");
  return BM_OK;
}
template <bool GROUPS, bool B_TR, int EPI>
bm_status launch_two_heights_cut(const GemmParams& p, hipStream_t st) {
  return p.K % BK ? launch_two_heights<GROUPS, B_TR, EPI, true>(p, st) : launch_two_heights<GROUPS, B_TR, EPI, false>(p, st);
}

template <bool CUT>
bm_status launch_parts(const TnParts& g, hipStream_t st) {
  constexpr size_t lds = (size_t)2 * (256 + 256) * BK * sizeof(bf16_t);
  auto kern = gemm_alt256_tn_parts_kernel<CUT>;
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_relaxed)) {
    BM_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_done.store(true, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(kern, dim3(g.wgs()), dim3(THREADS), lds, st, g);
  BM_CHECK_LAUNCH("gemm_alt_tn_parts");
  return BM_OK;
}

template <int SOURCE>
bm_status launch_source(const GemmParams& p, hipStream_t st) {
  constexpr size_t lds = (size_t)2 * (256 + 256) * BK * sizeof(bf16_t) + MOE_SOURCE_ROWS * sizeof(int32_t);
  static_assert(lds <= 160 * 1024, "the source rows lie behind the slices");
  auto kern = gemm_alt256_tn_source_kernel<SOURCE>;
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_relaxed)) {
    BM_CHECK_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    attr_done.store(true, std::memory_order_relaxed);
  }
  hipLaunchKernelGGL(kern, dim3(p.tiles_m * p.tiles_n * p.grid_groups), dim3(THREADS), lds, st, p);
  BM_CHECK_LAUNCH("gemm_alt_tn_source");
  return BM_OK;
}

template <int BM, int BN, bool A_TR, bool B_TR, int EPI>
bm_status launch_cut(const GemmParams& p, hipStream_t st) {
  if (p.K % BK) return launch_one<BM, BN, A_TR, B_TR, EPI, true>(p, st);
  return launch_one<BM, BN, A_TR, B_TR, EPI, false>(p, st);
}

template <int BM, int BN>
bm_status launch_tile(int layout, const GemmParams& p, hipStream_t st) {
  if (layout == GEMM_TN)
    return p.splits > 1 ? launch_cut<BM, BN, true, true, EPI_PARTIAL>(p, st) : launch_cut<BM, BN, true, true, EPI_ADD>(p, st);
  if (layout == GEMM_NT) {
    if (p.splits > 1) return launch_cut<BM, BN, false, false, EPI_PARTIAL>(p, st);
    // (256x128: N is a multiple of 256 there, so 128x256 tiles are never more and the plan takes them)
    if constexpr (BN == 256) if (p.swf_a) return launch_cut<BM, BN, false, false, EPI_SWIGLU_FWD>(p, st);
    return p.residual ? launch_cut<BM, BN, false, false, EPI_RES>(p, st) : launch_cut<BM, BN, false, false, EPI_PLAIN>(p, st);
  }
  if (p.splits > 1) return launch_cut<BM, BN, false, true, EPI_PARTIAL>(p, st);
  if (p.sw_up) return launch_cut<BM, BN, false, true, EPI_SWIGLU_BWD>(p, st);
  return p.residual ? launch_cut<BM, BN, false, true, EPI_RES>(p, st) : launch_cut<BM, BN, false, true, EPI_PLAIN>(p, st);
}

}  // namespace

bm_status launch_gemm_alt(int layout, int bm, int bn, const GemmParams& p, hipStream_t st) {
  if (bn == 128 && p.swf_a) { set_error("gemm: no SwiGLU forward on 256x128 tiles"); return BM_ERR_UNSUPPORTED; }
  if (bm == 256 && bn == 256) return launch_tile<256, 256>(layout, p, st);
  if (bm == 256 && bn == 128) return launch_tile<256, 128>(layout, p, st);
  return launch_tile<128, 256>(layout, p, st);
}

bm_status launch_gemm_alt_groups(int layout, const GemmParams& p, hipStream_t st) {
  if (layout == GEMM_NT)
    return p.swf_a ? launch_two_heights_cut<true, false, EPI_SWIGLU_FWD>(p, st) : launch_two_heights_cut<true, false, EPI_PLAIN>(p, st);
  return p.sw_up ? launch_two_heights_cut<true, true, EPI_SWIGLU_BWD>(p, st) : launch_two_heights_cut<true, true, EPI_PLAIN>(p, st);
}

bm_status launch_gemm_alt_mixed(int layout, const GemmParams& p, hipStream_t st) {
  if (layout == GEMM_NT) {
    if (p.swf_a) return launch_two_heights_cut<false, false, EPI_SWIGLU_FWD>(p, st);
    return p.residual ? launch_two_heights_cut<false, false, EPI_RES>(p, st) : launch_two_heights_cut<false, false, EPI_PLAIN>(p, st);
  }
  if (p.sw_up) return launch_two_heights_cut<false, true, EPI_SWIGLU_BWD>(p, st);
  return p.residual ? launch_two_heights_cut<false, true, EPI_RES>(p, st) : launch_two_heights_cut<false, true, EPI_PLAIN>(p, st);
}

bm_status launch_gemm_alt_tn_source(int operand, const GemmParams& p, hipStream_t st) {
  return operand == 0 ? launch_source<1>(p, st) : launch_source<2>(p, st);
}

bm_status launch_gemm_alt_tn_parts(const TnParts& g, hipStream_t st) {
  bool cut = false;
  for (int i = 0; i < g.n; ++i) cut = cut || g.part[i].K % BK;
  return cut ? launch_parts<true>(g, st) : launch_parts<false>(g, st);
}

}  // namespace bm
