"""The kernels in fp32 arithmetic at the edges of their variants (needs a GPU): both GEMM kernels and every block of
theirs with ragged edges, single elements and rows that are not aligned for wide loads; attention with eight lanes
per row and with one, also with a key that is not a number."""
import numpy as np
import pytest

import test_gpu_ops as ops
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

GEMM_CASES = [
    # M, N, K, extra columns of the operands
    (1, 1, 1, 0), (16, 16, 16, 0), (17, 15, 5, 0), (40, 192, 64, 0), (33, 70, 68, 4), (129, 47, 257, 3), (64, 16, 1000, 1),
    (1030, 1025, 36, 0), (1030, 1025, 35, 1),      # 2x2 blocks per wavefront, or tiles in LDS
    (2060, 2050, 20, 0), (2060, 2050, 33, 3),
    (700, 830, 45, 1), (830, 900, 100, 4),         # about a tile per CU
    (1000, 250, 1030, 1), (1000, 250, 1032, 0),    # k ranges
]


@pytest.mark.parametrize("dtype", [synth.DTYPE_BF16, synth.DTYPE_FP32], ids=["bf16", "fp32"])
@pytest.mark.parametrize("layout", [0, 1, 2], ids=["NT", "NN", "TN"])
@pytest.mark.parametrize("M,N,K,pad", GEMM_CASES)
def test_gemm(layout, dtype, M, N, K, pad):
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import to_device
    rng = np.random.default_rng(M + 3 * N + 7 * K + layout)
    a_shape, b_shape = (K, M) if layout == 2 else (M, K), (N, K) if layout == 0 else (K, N)
    A, B = (synth.to_storage(rng.standard_normal((r, c + pad), dtype=np.float32), dtype) for r, c in (a_shape, b_shape))
    A64, B64 = A[:, :a_shape[1]].astype(np.float64), B[:, :b_shape[1]].astype(np.float64)
    a, b = A64.T if layout == 2 else A64, B64.T if layout == 0 else B64
    C0 = rng.standard_normal((M, N), dtype=np.float32)
    fp32_out = layout == 2 or dtype == synth.DTYPE_FP32
    dC = torch.from_numpy(C0).cuda().to(torch.float32 if fp32_out else torch.bfloat16)
    nbytes = bm.gemm_scratch_bytes(layout, M, N, K, dtype)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    print(f"gemm layout={layout} dtype={dtype} M={M} N={N} K={K} pad={pad}", flush=True)
    bm.gemm(layout, dtype, M, N, K, to_device(A, dtype), A.shape[1], to_device(B, dtype), B.shape[1], dC, N, None, ws, nbytes)
    torch.cuda.synchronize()
    ref = a @ b + (C0 if layout == 2 else 0)
    # a sum of K products in fp32 in any order is off by at most (K + 1) roundings of sum |a b|; one more
    # for the accumulated C, and the rounding of a bf16 result
    bound = (K + 2) * 2.0 ** -24 * (np.abs(a) @ np.abs(b) + np.abs(C0)) + (0 if fp32_out else 2.0 ** -8 * np.abs(ref))
    assert (np.abs(dC.double().cpu().numpy() - ref) <= bound).all()


@pytest.mark.parametrize("dtype,Hq,Hkv,dh,lens,causal", [
    (synth.DTYPE_FP32, 4, 2, 8, [1, 31, 33, 15], 0), (synth.DTYPE_FP32, 4, 4, 32, [17, 130, 16], 1),
    (synth.DTYPE_FP32, 2, 1, 128, [70, 3], 1), (synth.DTYPE_FP32, 2, 2, 72, [65], 0),
    (synth.DTYPE_BF16, 4, 4, 16, [200, 7], 1),
    (synth.DTYPE_FP32, 16, 4, 16, [300, 1, 725], 1), (synth.DTYPE_FP32, 16, 16, 16, [129, 900], 0),   # one lane per row
])
def test_attention(dtype, Hq, Hkv, dh, lens, causal):
    ops.test_attention_matches_definition(dtype, Hq, Hkv, dh, lens, causal)


@pytest.mark.parametrize("dtype,Hq,Hkv,dh,lens,key,causal", [
    (synth.DTYPE_FP32, 4, 4, 16, [40, 33], 35, 0), (synth.DTYPE_FP32, 4, 2, 32, [70], 64, 1),   # the only key of its lane in the tile
    (synth.DTYPE_FP32, 2, 2, 72, [65], 0, 1), (synth.DTYPE_BF16, 4, 2, 16, [12, 36], 12 + 35, 0), (synth.DTYPE_FP32, 2, 1, 128, [33], 32, 1),
    (synth.DTYPE_FP32, 4, 4, 16, [40], 10, 0),                                                  # among others
    (synth.DTYPE_FP32, 16, 16, 16, [129, 900], 128, 0), (synth.DTYPE_FP32, 16, 4, 16, [1057], 1056, 1),   # one lane per row: alone in its tile
])
def test_a_nan_key_reaches_every_row_that_sees_it(dtype, Hq, Hkv, dh, lens, key, causal):
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import to_device
    rng = np.random.default_rng(sum(lens) + key)
    cu = synth.cu_from_lengths(lens)
    T, W = int(cu[-1]), (Hq + 2 * Hkv) * dh
    qkv = synth.to_storage(rng.standard_normal((T, W), dtype=np.float32), dtype)
    dqkv = to_device(qkv, dtype)
    dqkv[key, Hq * dh:(Hq + Hkv) * dh:dh] = float("nan")                 # one component of the key in every head
    o = torch.zeros((T, Hq * dh), dtype=dqkv.dtype, device="cuda")
    lse = torch.zeros((Hq, T), dtype=torch.float32, device="cuda")
    print(f"nan key dtype={dtype} Hq={Hq} Hkv={Hkv} dh={dh} lens={lens} key={key} causal={causal}", flush=True)
    bm.attention_forward(dtype, causal, Hq, Hkv, dh, dqkv, dqkv[:, Hq * dh:], dqkv[:, (Hq + Hkv) * dh:], W,
                         torch.from_numpy(cu).cuda(), cu, len(lens), T, max(lens), o, lse)
    torch.cuda.synchronize()
    rows = np.arange(T)
    s = np.searchsorted(cu, key, side="right") - 1
    sees = (rows >= (key if causal else cu[s])) & (rows < cu[s + 1])
    assert (np.isnan(o.float().cpu().numpy()).all(axis=1) == sees).all()
    assert (np.isfinite(lse.cpu().numpy()).all(axis=0) == ~sees).all()
