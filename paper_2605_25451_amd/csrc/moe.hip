// Routing, dispatch and combine kernels of the mixture-of-experts FFN.
//
// The paper's LLM backbone is a mixture-of-experts model (Sec. 4.1) and Sec. 3.3 names
// expert imbalance as a source of uneven operator times; it gives no arithmetic.  The
// reading built here: router logits = h W_r^T, probabilities = softmax over the experts,
// the k most probable experts are chosen (ties: lower index), their probabilities
// renormalised to sum 1 are the gates, no token is dropped.
//
// Dispatch layout.  The T*k routed rows are sorted by expert, token order inside an
// expert, and every expert's segment is padded to MOE_PAD rows, so a row block of the
// grouped GEMMs belongs to one expert.  The padded capacity T*k + E*(MOE_PAD-1), rounded
// up, is known on the host; everything data dependent (segment offsets, the row block ->
// expert table, the slot of each (token, choice)) stays on the device.  All counting is
// integer work in a fixed order, so the layout -- and with it every floating-point sum
// downstream -- is reproducible.
#include "common.h"

namespace bm {

namespace {

constexpr int MOE_MAX_E = 256;    // experts (4 logits per lane)
constexpr int MOE_MAX_K = 8;
constexpr int MOE_CHUNK = 256;    // tokens per workgroup in the counting kernels

// ---- router: softmax, top-k, gates (one wavefront per token) -------------------------
__global__ __launch_bounds__(256) void moe_route_kernel(const float* __restrict__ logits, int T, int E,
                                                        int k, float* __restrict__ probs,
                                                        int32_t* __restrict__ idx, float* __restrict__ gate) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + wave;
  if (t >= T) return;
  float v[4];
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int e = i * 64 + lane;
    v[i] = e < E ? logits[(size_t)t * E + e] : -INFINITY;
    mx = fmaxf(mx, v[i]);
  }
  mx = wave_max(mx);
  float p[4], s = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) { p[i] = (i * 64 + lane) < E ? expf(v[i] - mx) : 0.f; s += p[i]; }
  s = wave_sum(s);
  const float inv = 1.0f / s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    p[i] *= inv;
    const int e = i * 64 + lane;
    if (e < E) probs[(size_t)t * E + e] = p[i];
  }
  // k rounds of (largest logit, lowest index); a chosen logit is retired to -inf
  float sel[MOE_MAX_K];
  int who[MOE_MAX_K];
  float ssum = 0.f;
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    sel[j] = 0.f; who[j] = 0;
    if (j >= k) continue;
    float bv = -INFINITY; int be = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = i * 64 + lane;
      if (e < E && v[i] > bv) { bv = v[i]; be = e; }      // ascending e: the lower index wins a tie
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      const float ov = __shfl_xor(bv, off, WAVE);
      const int oe = __shfl_xor(be, off, WAVE);
      if (ov > bv || (ov == bv && oe < be)) { bv = ov; be = oe; }
    }
    // the owner retires it and everybody learns its probability
    float pw = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i * 64 + lane == be) { pw = p[i]; v[i] = -INFINITY; }
    pw = wave_sum(pw);
    sel[j] = pw; who[j] = be; ssum += pw;
  }
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j) {
      if (j < k) {
        idx[(size_t)t * k + j] = who[j];
        gate[(size_t)t * k + j] = sel[j] / ssum;
      }
    }
  }
}

// ---- dispatch layout ---------------------------------------------------------------------
__global__ __launch_bounds__(MOE_CHUNK) void moe_count_kernel(const int32_t* __restrict__ idx, int T, int E,
                                                              int k, int32_t* __restrict__ counts) {
  __shared__ int c[MOE_MAX_E];
  for (int e = threadIdx.x; e < MOE_MAX_E; e += MOE_CHUNK) c[e] = 0;
  __syncthreads();
  const int t = blockIdx.x * MOE_CHUNK + threadIdx.x;
  if (t < T)
    for (int j = 0; j < k; ++j) {
      const int e = idx[(size_t)t * k + j];
      if (e >= 0 && e < E) atomicAdd(&c[e], 1);           // integer count: order does not matter
    }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += MOE_CHUNK) counts[(size_t)blockIdx.x * E + e] = c[e];
}

// one workgroup: per expert the exclusive prefix over the token chunks, the padded segment
// offsets, and the row block -> expert table (-1 past the last segment).  Bound by latency, so no chain is longer than
// it has to be: eight counts of an expert are requested together, the offsets are a scan over the wavefronts, and an
// expert writes its own row blocks (one load after the other, one thread adding up and a search over the experts for every
// block took 41 us for 32 chunks of 128 experts; this takes 4.8).
__global__ __launch_bounds__(256) void moe_offsets_kernel(const int32_t* __restrict__ counts, int nblk, int E,
                                                          int32_t* __restrict__ base,
                                                          int32_t* __restrict__ expert_rows,
                                                          int32_t* __restrict__ tile_group, int n_tiles,
                                                          int32_t* __restrict__ row_tiles) {
  static_assert(MOE_MAX_E <= 256, "one thread per expert");
  __shared__ int wave_rows[4], wave_tiles[4];
  const int e = threadIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  int run = 0;
  if (e < E) {
    constexpr int AHEAD = 8;
    for (int b0 = 0; b0 < nblk; b0 += AHEAD) {
      int c[AHEAD];
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) c[i] = b0 + i < nblk ? counts[(size_t)(b0 + i) * E + e] : 0;
#pragma unroll
      for (int i = 0; i < AHEAD; ++i) {
        if (b0 + i < nblk) base[(size_t)(b0 + i) * E + e] = run;
        run += c[i];
      }
    }
  }
  const int padded = (run + MOE_PAD - 1) / MOE_PAD * MOE_PAD;
  const int own_tiles = (padded / MOE_PAD + 1) / 2;       // of two row blocks, the last of one where they are odd
  int sum = padded, tiles = own_tiles;                    // inclusive over the wavefront
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int below = __shfl_up(sum, off, WAVE), tiles_below = __shfl_up(tiles, off, WAVE);
    if (lane >= off) { sum += below; tiles += tiles_below; }
  }
  if (lane == 63) { wave_rows[wave] = sum; wave_tiles[wave] = tiles; }
  __syncthreads();
  int start = sum - padded, all = 0, tile0 = tiles - own_tiles, all_tiles = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    if (w < wave) { start += wave_rows[w]; tile0 += wave_tiles[w]; }
    all += wave_rows[w]; all_tiles += wave_tiles[w];
  }
  if (e == 0) row_tiles[0] = all_tiles;
  for (int t = 0; t < own_tiles; ++t)
    row_tiles[1 + tile0 + t] = 2 * (start / MOE_PAD + 2 * t) + (2 * t + 1 < padded / MOE_PAD ? 1 : 0);
  if (e < E) {
    expert_rows[e] = start;
    for (int tile = start / MOE_PAD; tile < (start + padded) / MOE_PAD && tile < n_tiles; ++tile) tile_group[tile] = e;
  }
  if (e == 0) expert_rows[E] = all;
  for (int tile = all / MOE_PAD + threadIdx.x; tile < n_tiles; tile += 256) tile_group[tile] = -1;
}

// rows that fill up a segment have no token and no weight
__global__ void moe_clear_rows_kernel(int32_t* __restrict__ row_token, float* __restrict__ row_gate, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) { row_token[i] = -1; row_gate[i] = 0.f; }
}

// slot of every (token, choice): segment offset + tokens of earlier chunks + rank inside the
// chunk (token order); also the inverse tables row -> token and row -> gate
__global__ __launch_bounds__(MOE_CHUNK) void moe_slot_kernel(
    const int32_t* __restrict__ idx, const float* __restrict__ gate, int T, int E, int k,
    const int32_t* __restrict__ base, const int32_t* __restrict__ expert_rows,
    int32_t* __restrict__ slot, int32_t* __restrict__ row_token, float* __restrict__ row_gate, int cap) {
  __shared__ unsigned long long chosen[MOE_CHUNK / 64][MOE_MAX_E];   // the lanes of a wavefront that chose an expert
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = blockIdx.x * MOE_CHUNK + threadIdx.x;
  // (a bit per lane, or-ed into LDS, instead of a ballot per expert: 28 -> 9.5 us at 8192 tokens, 128 experts, 8 choices)
  for (int e = lane; e < E; e += WAVE) chosen[wave][e] = 0ull;
  __syncthreads();
  int mine[MOE_MAX_K];
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    mine[j] = (t < T && j < k) ? idx[(size_t)t * k + j] : -1;
    if (mine[j] >= 0 && mine[j] < E) atomicOr(&chosen[wave][mine[j]], 1ull << lane);
  }
  const unsigned long long below = (1ull << lane) - 1ull;
  __syncthreads();
  if (t >= T) return;
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    const int e = mine[j];
    if (j >= k || e < 0 || e >= E) continue;
    int r = __popcll(chosen[wave][e] & below);
    for (int w = 0; w < wave; ++w) r += __popcll(chosen[w][e]);
    const int s = expert_rows[e] + base[(size_t)blockIdx.x * E + e] + r;
    slot[(size_t)t * k + j] = s;
    if (s >= 0 && s < cap) {
      row_token[s] = t;
      row_gate[s] = gate[(size_t)t * k + j];
    }
  }
}

// ---- row movement ------------------------------------------------------------------------------
// dst[row] = scale(row) * src[row_token[row]]  (zeros for padding rows); scale = row_gate or 1.  A thread per 16 bytes.
template <typename T>
__global__ void moe_gather_chunks_kernel(const T* __restrict__ src, const int32_t* __restrict__ row_token,
                                         const float* __restrict__ row_gate, T* __restrict__ dst, int rows,
                                         int d, int n_src) {
  constexpr int VEC = Elt<T>::VEC;
  const int per = d / VEC;
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long)rows * per) return;
  const int row = (int)(gid / per), c = (int)(gid % per) * VEC;
  const int t = row_token[row];
  float v[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) v[e] = 0.f;
  if (t >= 0 && t < n_src) {
    load16(src + (size_t)t * d + c, v);
    if (row_gate) {
      const float g = row_gate[row];
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[e] *= g;
    }
  }
  store16(dst + (size_t)row * d + c, v);
}

// A wavefront per row: its token is looked up once and its loads are in flight together (82000 x 2048 bf16 92 -> 83 us, 4.5 TB/s),
// but lanes that the last 64 chunks of 16 bytes do not fill are idle; see moe_gather for the line between the two.
template <typename T>
__global__ __launch_bounds__(256) void moe_gather_rows_kernel(const T* __restrict__ src, const int32_t* __restrict__ row_token,
                                                              const float* __restrict__ row_gate, T* __restrict__ dst,
                                                              int rows, int d, int n_src) {
  constexpr int VEC = Elt<T>::VEC, AHEAD = 4;
  const int lane = threadIdx.x & 63;
  const int row = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
  if (row >= rows) return;
  const int t = row_token[row];
  const bool live = t >= 0 && t < n_src;
  const bool scaled = live && row_gate;
  const float g = scaled ? row_gate[row] : 1.f;
  const T* from = src + (size_t)(live ? t : 0) * d;
  T* to = dst + (size_t)row * d;
  for (int c0 = lane * VEC; c0 < d; c0 += AHEAD * WAVE * VEC) {
    float v[AHEAD][VEC];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) v[i][e] = 0.f;
      const int c = c0 + i * WAVE * VEC;
      if (live && c < d) load16(from + c, v[i]);
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
      const int c = c0 + i * WAVE * VEC;
      if (scaled)
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[i][e] *= g;
      if (c < d) store16(to + c, v[i]);
    }
  }
}

// out[t] = (res ? res[t] : 0) + sum_j w(t,j) * rows[slot[t,j]],  w = gate or 1; choices in order
template <typename T>
__global__ void moe_combine_kernel(const T* __restrict__ rows, const int32_t* __restrict__ slot,
                                   const float* __restrict__ gate, const T* __restrict__ res,
                                   T* __restrict__ out, int Tn, int k, int d, int cap) {
  constexpr int VEC = Elt<T>::VEC;
  const int per = d / VEC;
  const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (long)Tn * per) return;
  const int t = (int)(gid / per), c = (int)(gid % per) * VEC;
  float acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) acc[e] = 0.f;
  for (int j = 0; j < k; ++j) {
    const int s = slot[(size_t)t * k + j];
    if (s < 0 || s >= cap) continue;
    float v[VEC];
    load16(rows + (size_t)s * d + c, v);
    const float g = gate ? gate[(size_t)t * k + j] : 1.0f;
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] = fmaf(g, v[e], acc[e]);
  }
  if (res) {
    float r[VEC];
    load16(res + (size_t)t * d + c, r);
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[e] += r[e];
  }
  store16(out + (size_t)t * d + c, acc);
}

// ---- router backward (one wavefront per token) ------------------------------------------------
// dgate[t,j] = <dm[t], y_rows[slot[t,j]]>; then through the gate normalisation and the
// softmax: dlogit_e = p_e (dp_e - sum_e' p_e' dp_e'), dp nonzero on the chosen experts only.
// <dm, y> = <dm W_down, a>, which the SwiGLU backward's epilogue has in registers: with its partial sums (row_dot) 65536 rows
// of 2048 columns are not read (96 -> 14 us)
template <typename T>
__global__ __launch_bounds__(256) void moe_router_bwd_kernel(
    const T* __restrict__ dm, const T* __restrict__ y_rows, const float* __restrict__ row_dot, int parts,
    const int32_t* __restrict__ slot, const int32_t* __restrict__ idx, const float* __restrict__ gate,
    const float* __restrict__ probs, T* __restrict__ dlogits, int Tn, int E, int k, int d, int cap) {
  constexpr int VEC = Elt<T>::VEC;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + wave;
  if (t >= Tn) return;
  float dg[MOE_MAX_K];
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    dg[j] = 0.f;
    if (j >= k) continue;
    const int s = slot[(size_t)t * k + j];
    if (s < 0 || s >= cap) continue;
    float part = 0.f;
    if (row_dot)
      for (int c = lane; c < parts; c += WAVE) part += row_dot[(size_t)s * parts + c];
    else for (int c = lane * VEC; c < d; c += WAVE * VEC) {
      float a[VEC], b[VEC];
      load16(dm + (size_t)t * d + c, a);
      load16(y_rows + (size_t)s * d + c, b);
#pragma unroll
      for (int e = 0; e < VEC; ++e) part = fmaf(a[e], b[e], part);
    }
    dg[j] = wave_sum(part);
  }
  float ssum = 0.f, dot_g = 0.f;
  int who[MOE_MAX_K];
  float ps[MOE_MAX_K];
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    who[j] = -1; ps[j] = 0.f;
    if (j >= k) continue;
    who[j] = idx[(size_t)t * k + j];
    ps[j] = probs[(size_t)t * E + who[j]];
    ssum += ps[j];
    dot_g += dg[j] * gate[(size_t)t * k + j];
  }
  float dsel[MOE_MAX_K], dot_p = 0.f;
#pragma unroll
  for (int j = 0; j < MOE_MAX_K; ++j) {
    dsel[j] = j < k ? (dg[j] - dot_g) / ssum : 0.f;
    dot_p += ps[j] * dsel[j];
  }
  for (int e = lane; e < E; e += WAVE) {
    float dp = 0.f;
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j)
      if (who[j] == e) dp = dsel[j];
    dlogits[(size_t)t * E + e] = Elt<T>::from_f(probs[(size_t)t * E + e] * (dp - dot_p));
  }
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
int moe_row_capacity(int T, int E, int k) {
  const long r = (long)T * k + (long)E * (MOE_PAD - 1);
  return (int)((r + MOE_PAD - 1) / MOE_PAD * MOE_PAD);
}

size_t moe_layout_scratch_bytes(int T, int E) {
  const size_t nblk = (size_t)cdiv(T, MOE_CHUNK);
  return 2 * align_up(nblk * E * sizeof(int32_t), 256);      // counts + base
}

bm_status moe_check(int E, int k, int d, int dtype) {
  if (E < 1 || E > MOE_MAX_E) { set_error("moe: %d experts outside [1,%d]", E, MOE_MAX_E); return BM_ERR_UNSUPPORTED; }
  if (k < 1 || k > MOE_MAX_K || k > E) { set_error("moe: top_k %d outside [1,min(%d,E)]", k, MOE_MAX_K); return BM_ERR_UNSUPPORTED; }
  const int vec = dtype == BM_DTYPE_BF16 ? 8 : 4;
  if (d % vec) { set_error("moe: hidden %d not a multiple of %d", d, vec); return BM_ERR_UNSUPPORTED; }
  return BM_OK;
}

bm_status moe_route(const float* logits, int T, int E, int k, float* probs, int32_t* idx, float* gate,
                    hipStream_t st) {
  hipLaunchKernelGGL(moe_route_kernel, dim3(cdiv(T, 4)), dim3(256), 0, st, logits, T, E, k, probs, idx, gate);
  BM_CHECK_LAUNCH("moe_route");
  return BM_OK;
}

bm_status moe_layout(const MoeTables& m, int T, int E, int k, void* scratch, hipStream_t st) {
  const int nblk = cdiv(T, MOE_CHUNK);
  int32_t* counts = (int32_t*)scratch;
  int32_t* base = (int32_t*)((char*)scratch + align_up((size_t)nblk * E * sizeof(int32_t), 256));
  hipLaunchKernelGGL(moe_count_kernel, dim3(nblk), dim3(MOE_CHUNK), 0, st, m.idx, T, E, k, counts);
  hipLaunchKernelGGL(moe_offsets_kernel, dim3(1), dim3(256), 0, st, counts, nblk, E, base, m.expert_rows,
                     m.tile_group, m.cap / MOE_PAD, m.row_tiles);
  hipLaunchKernelGGL(moe_clear_rows_kernel, dim3(cdiv(m.cap, 256)), dim3(256), 0, st, m.row_token, m.row_gate, m.cap);
  hipLaunchKernelGGL(moe_slot_kernel, dim3(nblk), dim3(MOE_CHUNK), 0, st, m.idx, m.gate, T, E, k, base,
                     m.expert_rows, m.slot, m.row_token, m.row_gate, m.cap);
  BM_CHECK_LAUNCH("moe_layout");
  return BM_OK;
}

// A wavefront per row where rows fill their trips of 64 lanes or are at least three trips long.  us, 16-byte chunks / rows, 36000 rows of
// bf16: 64 columns 3.8 / 7.7, 128 5.2 / 8.3, 256 7.2 / 8.9, 320 8.1 / 9.4, 512 12.4 / 11.6, 640 13.6 / 14.4, 1024 23.9 / 20.6, 1088 22.0 / 22.3,
// 2048 44.7 / 41.0; 20000 rows: 1216 13.8 / 14.2, 1600 20.2 / 18.3, 2880 35.6 / 33.1, 4160 48.8 / 47.1.
bm_status moe_gather(int dtype, const void* src, const MoeTables& m, int use_gate, void* dst, int d, int T,
                     hipStream_t st) {
  const float* rg = use_gate ? m.row_gate : nullptr;
  const int chunks = d / (dtype == BM_DTYPE_BF16 ? 8 : 4);
  const bool by_rows = chunks % WAVE == 0 || chunks >= 3 * WAVE;
  const dim3 grid(by_rows ? cdiv(m.cap, 4) : cdiv((long)m.cap * chunks, 256));
  if (dtype == BM_DTYPE_BF16)
    hipLaunchKernelGGL(by_rows ? moe_gather_rows_kernel<bf16_t> : moe_gather_chunks_kernel<bf16_t>, grid, dim3(256), 0, st,
                       (const bf16_t*)src, m.row_token, rg, (bf16_t*)dst, m.cap, d, T);
  else
    hipLaunchKernelGGL(by_rows ? moe_gather_rows_kernel<float> : moe_gather_chunks_kernel<float>, grid, dim3(256), 0, st,
                       (const float*)src, m.row_token, rg, (float*)dst, m.cap, d, T);
  BM_CHECK_LAUNCH("moe_gather");
  return BM_OK;
}

bm_status moe_combine(int dtype, const void* rows, const MoeTables& m, int use_gate, const void* res,
                      void* out, int T, int k, int d, hipStream_t st) {
  const int vec = dtype == BM_DTYPE_BF16 ? 8 : 4;
  const long n = (long)T * (d / vec);
  const float* g = use_gate ? m.gate : nullptr;
  if (dtype == BM_DTYPE_BF16)
    hipLaunchKernelGGL(moe_combine_kernel<bf16_t>, dim3(cdiv(n, 256)), dim3(256), 0, st, (const bf16_t*)rows,
                       m.slot, g, (const bf16_t*)res, (bf16_t*)out, T, k, d, m.cap);
  else
    hipLaunchKernelGGL(moe_combine_kernel<float>, dim3(cdiv(n, 256)), dim3(256), 0, st, (const float*)rows,
                       m.slot, g, (const float*)res, (float*)out, T, k, d, m.cap);
  BM_CHECK_LAUNCH("moe_combine");
  return BM_OK;
}

bm_status moe_router_backward(int dtype, const void* dm, const void* y_rows, const float* row_dot, int parts, const MoeTables& m,
                              void* dlogits, int T, int E, int k, int d, hipStream_t st) {
  if (dtype == BM_DTYPE_BF16)
    hipLaunchKernelGGL(moe_router_bwd_kernel<bf16_t>, dim3(cdiv(T, 4)), dim3(256), 0, st, (const bf16_t*)dm,
                       (const bf16_t*)y_rows, row_dot, parts, m.slot, m.idx, m.gate, m.probs, (bf16_t*)dlogits, T, E, k, d, m.cap);
  else
    hipLaunchKernelGGL(moe_router_bwd_kernel<float>, dim3(cdiv(T, 4)), dim3(256), 0, st, (const float*)dm,
                       (const float*)y_rows, row_dot, parts, m.slot, m.idx, m.gate, m.probs, (float*)dlogits, T, E, k, d, m.cap);
  BM_CHECK_LAUNCH("moe_router_backward");
  return BM_OK;
}

}  // namespace bm
