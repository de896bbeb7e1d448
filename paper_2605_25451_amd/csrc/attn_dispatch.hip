// Attention back-end selection: MFMA flash kernels for bf16 with head sizes
// they cover, the generic fp32-arithmetic kernels otherwise.
#include "common.h"

namespace bm {

bool attention_mfma_supported(const AttnArgs& a);
bm_status attention_forward_mfma(const AttnArgs& a, void* o, float* lse, hipStream_t st);
void attention_mfma_plan(const AttnArgs& a, int* fwd_rows, int* dq_rows, int* dkdv_rows);
void attention_mfma_backward_plan(const AttnArgs& a, int* launches, int* dkdv_wgs, int* dq_wgs);
size_t attention_backward_mfma_scratch_bytes(int Hq, int Hkv, int dh, int Tq, int Tk);
bm_status attention_backward_mfma(const AttnArgs& a, const void* o, const void* d_o, const float* lse,
                                  void* dq, void* dk, void* dv, int ld_dqkv, void* scratch,
                                  size_t scratch_bytes, hipStream_t st);

// unmasked (query, key) pairs inside the sequences
static double attn_pairs(const AttnArgs& a) {
  double pairs = 0;
  const int32_t* ck = a.kv_cu_host();
  for (int s = 0; s < a.S; ++s) {
    double L = a.cu_host[s + 1] - a.cu_host[s], Lk = ck[s + 1] - ck[s];
    pairs += a.causal ? L * (L + 1) / 2 : L * Lk;
  }
  return pairs;
}

bm_status attention_forward(const AttnArgs& a, void* o, float* lse, hipStream_t st) {
  ProfScope prof(PROF_ATTN_FWD, 4.0 * a.dh * a.Hq * attn_pairs(a), st);
  if (attention_mfma_supported(a)) return attention_forward_mfma(a, o, lse, st);
  return attention_forward_generic(a, o, lse, st);
}

size_t attention_backward_scratch_bytes(int Hq, int Hkv, int dh, int Tq, int Tk) {
  size_t generic = align_up((size_t)Hq * Tq * sizeof(float), 256);   // delta
  size_t mfma = attention_backward_mfma_scratch_bytes(Hq, Hkv, dh, Tq, Tk);
  return generic > mfma ? generic : mfma;
}

size_t attention_backward_scratch_bytes(int Hq, int Hkv, int dh, int T) {
  return attention_backward_scratch_bytes(Hq, Hkv, dh, T, T);
}

// does a gradient's memory, first to last row, touch an input's?
static bool in_place(const AttnArgs& a, const void* o, const void* d_o, const void* dq, const void* dk, const void* dv,
                     int ld_dqkv) {
  struct Span { uintptr_t begin, end; };
  auto span = [&](const void* p, int rows, int ld, int heads) {
    const uintptr_t b = reinterpret_cast<uintptr_t>(p);
    return Span{b, rows > 0 ? b + ((size_t)(rows - 1) * ld + (size_t)heads * a.dh) * elt_size(a.dtype) : b};
  };
  const int wide = a.Hq * a.dh, ld_dkv = a.ld_dkv ? a.ld_dkv : ld_dqkv;
  const Span in[] = {span(a.q, a.T, a.ld_qkv, a.Hq), span(o, a.T, wide, a.Hq), span(d_o, a.T, wide, a.Hq),
                     span(a.k, a.kv_T(), a.kv_ld(), a.Hkv), span(a.v, a.kv_T(), a.kv_ld(), a.Hkv)};
  const Span out[] = {span(dq, a.T, ld_dqkv, a.Hq), span(dk, a.kv_T(), ld_dkv, a.Hkv), span(dv, a.kv_T(), ld_dkv, a.Hkv)};
  for (const Span& x : in)
    for (const Span& y : out)
      if (x.begin < y.end && y.begin < x.end) return true;
  return false;
}

bm_status attention_backward(const AttnArgs& args, const void* o, const void* d_o, const float* lse,
                             void* dq, void* dk, void* dv, int ld_dqkv, void* scratch,
                             size_t scratch_bytes, hipStream_t st) {
  AttnArgs a = args;
  a.in_place = in_place(a, o, d_o, dq, dk, dv, ld_dqkv);
  ProfScope prof(PROF_ATTN_BWD, 10.0 * a.dh * a.Hq * attn_pairs(a), st);
  if (attention_mfma_supported(a))
    return attention_backward_mfma(a, o, d_o, lse, dq, dk, dv, ld_dqkv, scratch, scratch_bytes, st);
  return attention_backward_generic(a, o, d_o, lse, dq, dk, dv, ld_dqkv, (float*)scratch, st);
}

}  // namespace bm

using namespace bm;

static bm_status probe_args(int32_t mask, int32_t Hq, int32_t Hkv, int32_t dh, const int32_t* cu_q_host, const int32_t* cu_k_host,
                            int32_t S, AttnArgs* a) {
  BM_ARG_CHECK(mask == 0 || mask == 1, "attention plan: mask %d", mask);
  BM_ARG_CHECK(Hq > 0 && Hkv > 0 && dh > 0 && Hq % Hkv == 0, "attention plan: bad head counts %d/%d", Hq, Hkv);
  BM_ARG_CHECK(S >= 1 && cu_q_host, "attention plan: NULL offsets or no sequence");
  a->dtype = BM_DTYPE_BF16; a->causal = mask; a->Hq = Hq; a->Hkv = Hkv; a->dh = dh; a->S = S;
  a->ld_qkv = (Hq + 2 * Hkv) * dh;
  a->cu_host = cu_q_host; a->T = cu_q_host[S];
  static const int32_t on_device = 0;               // only says that the keys have a packing of their own
  if (cu_k_host) { a->cu_k_dev = &on_device; a->cu_k_host = cu_k_host; a->Tk = cu_k_host[S]; a->ld_kv = a->ld_qkv; }
  return BM_OK;
}

extern "C" bm_status bm_probe_attention_plan(int32_t mask, int32_t Hq, int32_t Hkv, int32_t dh, const int32_t* cu_q_host,
                                             const int32_t* cu_k_host, int32_t S, int32_t* fwd_rows, int32_t* dq_rows,
                                             int32_t* dkdv_rows) {
  BM_ARG_CHECK(fwd_rows && dq_rows && dkdv_rows, "bm_probe_attention_plan: NULL pointer");
  AttnArgs a{};
  BM_RETURN_IF(probe_args(mask, Hq, Hkv, dh, cu_q_host, cu_k_host, S, &a));
  *fwd_rows = *dq_rows = *dkdv_rows = 0;
  if (attention_mfma_supported(a)) attention_mfma_plan(a, fwd_rows, dq_rows, dkdv_rows);
  return BM_OK;
}

extern "C" bm_status bm_probe_attention_backward_plan(int32_t mask, int32_t Hq, int32_t Hkv, int32_t dh, const int32_t* cu_q_host,
                                                      const int32_t* cu_k_host, int32_t S, int32_t* launches,
                                                      int32_t* dkdv_wgs, int32_t* dq_wgs) {
  BM_ARG_CHECK(launches && dkdv_wgs && dq_wgs, "bm_probe_attention_backward_plan: NULL pointer");
  AttnArgs a{};
  BM_RETURN_IF(probe_args(mask, Hq, Hkv, dh, cu_q_host, cu_k_host, S, &a));
  *launches = *dkdv_wgs = *dq_wgs = 0;
  if (attention_mfma_supported(a)) attention_mfma_backward_plan(a, launches, dkdv_wgs, dq_wgs);
  return BM_OK;
}
