"""GEMM parity at the edges of the tiles and of the k split (needs a GPU): every tile the plan knows, with
ragged rows, columns and contractions, few rows against a long contraction, and a product that is given
no workspace to split in.  Tolerances are those of the other GEMM tests (bf16 storage of the result
2e-2, fp32 weight gradient 1e-4)."""
import numpy as np
import pytest

from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # layout, M, N, K
    (0, 5477, 1024, 1024), (1, 5477, 1024, 1016), (0, 1032, 5480, 1024), (1, 1032, 5480, 584),   # 128 x 256 and 256 x 128
    (0, 2049, 4104, 64), (0, 2049, 4104, 120), (1, 2049, 4104, 136), (1, 2049, 4104, 200),       # 256 x 256: 1 to 4 slices, cut
    (2, 4104, 2056, 1), (2, 4104, 2056, 65), (2, 4104, 2056, 129), (2, 4104, 2056, 777),
    (0, 577, 1024, 4096), (1, 577, 1032, 4104), (0, 1, 1024, 4096), (1, 40, 1024, 11008), (0, 300, 2048, 2056),   # split
    (2, 1024, 1032, 5477), (2, 264, 256, 4001),
]


@pytest.mark.parametrize("scratch", [True, False], ids=["workspace", "no-workspace"])
@pytest.mark.parametrize("layout,M,N,K", CASES)
def test_gemm_tiles(layout, M, N, K, scratch):
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import to_device
    if not scratch and (layout == 2 or M < 577):
        pytest.skip("weight gradients and skinny products are given the workspace they ask for")
    rng = np.random.default_rng(M + 3 * N + 7 * K + layout)
    A = synth.round_to_bf16(rng.standard_normal((K, M) if layout == 2 else (M, K), dtype=np.float32))
    B = synth.round_to_bf16(rng.standard_normal((N, K) if layout == 0 else (K, N), dtype=np.float32))
    bias = None if layout == 2 else synth.round_to_bf16(rng.standard_normal(N, dtype=np.float32))
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    dA, dB = to_device(A, synth.DTYPE_BF16), to_device(B, synth.DTYPE_BF16)
    if layout == 2:
        C0 = rng.standard_normal((M, N), dtype=np.float32)
        ref, dC = C0 + A64.T @ B64, torch.from_numpy(C0).cuda()
    else:
        ref = A64 @ (B64.T if layout == 0 else B64) + bias
        dC = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    nbytes = bm.gemm_scratch_bytes(layout, M, N, K, synth.DTYPE_BF16) if scratch else 0
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    print(f"gemm layout={layout} M={M} N={N} K={K} scratch={nbytes}", flush=True)
    bm.gemm(layout, synth.DTYPE_BF16, M, N, K, dA, A.shape[1], dB, B.shape[1], dC, N,
            None if bias is None else to_device(bias, synth.DTYPE_BF16), ws if nbytes else None, nbytes)
    torch.cuda.synchronize()
    got = dC.double().cpu().numpy()
    assert np.abs(got - ref).max() <= (1e-4 if layout == 2 else 2e-2) * np.abs(ref).max()


@pytest.mark.parametrize("layout,M,N,K", [
    (0, 2049, 4104, 72), (0, 2049, 4104, 184), (1, 2049, 4104, 88), (0, 1032, 5480, 120), (1, 1032, 5480, 136),
    (2, 4104, 2056, 71), (2, 4104, 2056, 95), (2, 2056, 4104, 129), (2, 4104, 2056, 190), (2, 1032, 5480, 76), (2, 5480, 1032, 67),
])
def test_cut_slices(layout, M, N, K):
    """Contractions that end inside a slice: what memory holds behind them (here: not a number) stays out of the sums."""
    import torch
    from paper_2605_25451_amd import binding as bm
    rng = np.random.default_rng(M + 3 * N + 7 * K + layout)
    a_shape, b_shape = (K, M) if layout == 2 else (M, K), (N, K) if layout == 0 else (K, N)
    A, B = (synth.round_to_bf16(rng.standard_normal(s, dtype=np.float32)) for s in (a_shape, b_shape))

    def padded(a, rows, cols):
        t = torch.full((a.shape[0] + rows, a.shape[1] + cols), float("nan"), dtype=torch.bfloat16, device="cuda")
        t[:a.shape[0], :a.shape[1]] = torch.from_numpy(a).cuda()
        return t
    dA = padded(A, *((64, 0) if layout == 2 else (0, 64)))
    dB = padded(B, *((0, 64) if layout == 0 else (64, 0)))
    a, b = (A.T if layout == 2 else A).astype(np.float64), (B.T if layout == 0 else B).astype(np.float64)
    dC = torch.zeros((M, N), dtype=torch.float32 if layout == 2 else torch.bfloat16, device="cuda")
    nbytes = bm.gemm_scratch_bytes(layout, M, N, K, synth.DTYPE_BF16)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    print(f"gemm cut layout={layout} M={M} N={N} K={K}", flush=True)
    bm.gemm(layout, synth.DTYPE_BF16, M, N, K, dA, dA.shape[1], dB, dB.shape[1], dC, N, None, ws, nbytes)
    torch.cuda.synchronize()
    ref = a @ b
    # at most K + 1 roundings of fp32 in any order of the sum, and the rounding of a bf16 result
    bound = (K + 1) * 2.0 ** -24 * (np.abs(a) @ np.abs(b)) + (0 if layout == 2 else 2.0 ** -8 * np.abs(ref))
    assert (np.abs(dC.double().cpu().numpy() - ref) <= bound).all()
