"""GEMM parity at the edges of the tiles and of the k split (needs a GPU): every tile the plan knows in every layout,
with ragged rows, columns and contractions, few rows against a long contraction, and a product that is given
no workspace to split in.  The plan of each case is asserted, so that another choice of tiles cannot drop a
kernel from this file."""
import numpy as np
import pytest

from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

T256, T128x256, T256x128, T128 = (256, 256), (128, 256), (256, 128), (128, 128)
CASES = [
    # layout, M, N, K, tile, k range split
    (0, 2049, 4104, 64, T256, False), (0, 2049, 4104, 184, T256, False), (1, 2049, 4104, 136, T256, False),   # 1 to 4 slices, cut
    (1, 2049, 4104, 200, T256, False), (2, 2976, 2960, 640, T256, False), (2, 1704, 4640, 808, T256, False),
    (0, 932, 5288, 448, T128x256, False), (0, 8273, 656, 456, T128x256, False), (1, 1466, 5272, 256, T128x256, False),
    (1, 7117, 648, 520, T128x256, False), (2, 4672, 1160, 1256, T128x256, False),
    (0, 2960, 2096, 320, T256x128, False), (0, 4339, 1312, 456, T256x128, False), (1, 1187, 4896, 320, T256x128, False),
    (1, 6004, 800, 568, T256x128, False), (2, 2752, 2088, 1224, T256x128, False), (2, 4568, 1040, 1473, T256x128, False),
    (2, 4104, 2056, 1, (0, 0), False), (2, 4104, 2056, 65, T128, False), (2, 4104, 2056, 129, T128, False), (2, 4104, 2056, 777, T256, False),
    (0, 5477, 1024, 1024, T128x256, False), (1, 5477, 1024, 1016, T128x256, False), (0, 1032, 5480, 1024, T128x256, False),
    (1, 1032, 5480, 584, T128x256, False),
    # split
    (0, 577, 1024, 4096, T128, True), (1, 577, 1032, 4104, T128, True), (0, 1, 1024, 4096, T128, True), (1, 40, 1024, 11008, T128, True),
    (0, 300, 2048, 2056, T128, True), (2, 264, 256, 4001, T128, True),
    (0, 2, 4856, 4288, T128x256, True), (0, 1, 5280, 5968, T128x256, True), (1, 2, 5264, 6848, T128x256, True), (1, 1, 3736, 8536, T128x256, True),
    (0, 129, 3640, 8032, T256x128, True), (1, 142, 4384, 4472, T256x128, True),
    (2, 64, 5544, 7545, T128x256, True), (2, 264, 3920, 4087, T128x256, True), (2, 152, 4448, 8451, T256x128, True), (2, 1024, 1032, 5477, T128, True),
    (2, 3696, 672, 8923, T256, True),
]


@pytest.mark.parametrize("scratch", [True, False], ids=["workspace", "no-workspace"])
@pytest.mark.parametrize("layout,M,N,K,tile,split", CASES)
def test_gemm_tiles(layout, M, N, K, tile, split, scratch):
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import to_device
    if not scratch and (layout == 2 or M < 577):
        pytest.skip("weight gradients and skinny products are given the workspace they ask for")
    if scratch:
        plan = bm.probe_gemm_plan(layout, M, N, K)
        assert plan[:2] == tile and (plan[2] > 1) == split, plan
    rng = np.random.default_rng(M + 3 * N + 7 * K + layout)
    A = synth.round_to_bf16(rng.standard_normal((K, M) if layout == 2 else (M, K), dtype=np.float32))
    B = synth.round_to_bf16(rng.standard_normal((N, K) if layout == 0 else (K, N), dtype=np.float32))
    bias = None if layout == 2 else synth.round_to_bf16(rng.standard_normal(N, dtype=np.float32))
    A64, B64 = A.astype(np.float64), B.astype(np.float64)
    a, b = A64.T if layout == 2 else A64, B64.T if layout == 0 else B64
    dA, dB = to_device(A, synth.DTYPE_BF16), to_device(B, synth.DTYPE_BF16)
    if layout == 2:
        start = rng.standard_normal((M, N), dtype=np.float32)
        dC = torch.from_numpy(start).cuda()
    else:
        start = bias
        dC = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    ref = a @ b + start
    nbytes = bm.gemm_scratch_bytes(layout, M, N, K, synth.DTYPE_BF16) if scratch else 0
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    print(f"gemm layout={layout} M={M} N={N} K={K} scratch={nbytes}", flush=True)
    bm.gemm(layout, synth.DTYPE_BF16, M, N, K, dA, A.shape[1], dB, B.shape[1], dC, N,
            None if bias is None else to_device(bias, synth.DTYPE_BF16), ws if nbytes else None, nbytes)
    torch.cuda.synchronize()
    # a sum of K products in fp32 in any order, and the bias or the old C: at most K + 2 roundings of the
    # sum of absolute values; and the rounding of a bf16 result
    bound = (K + 2) * 2.0 ** -24 * (np.abs(a) @ np.abs(b) + np.abs(start)) + (0 if layout == 2 else 2.0 ** -8 * np.abs(ref))
    assert (np.abs(dC.double().cpu().numpy() - ref) <= bound).all()


@pytest.mark.parametrize("layout,M,N,K", [
    (0, 2049, 4104, 184), (1, 1700, 4704, 136), (2, 1432, 5424, 391), (2, 2776, 2976, 456),         # 256 x 256
    (0, 8273, 656, 456), (1, 7117, 648, 520), (2, 1040, 4568, 1473),                               # 128 x 256
    (0, 4339, 1312, 456), (1, 3637, 1848, 400), (2, 4568, 1040, 1473),                              # 256 x 128
    (0, 1032, 5480, 72), (1, 1032, 5480, 88), (2, 4104, 2056, 71), (2, 2056, 4104, 95),             # 128 x 128
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


def test_a_workspace_that_is_not_aligned_is_left_alone():
    import torch
    from paper_2605_25451_amd import binding as bm
    M, N, K = 577, 1024, 4096
    gen = torch.Generator(device="cuda").manual_seed(1)
    A, B = (torch.randn(s, device="cuda", generator=gen).bfloat16() for s in ((M, K), (N, K)))
    nbytes = bm.gemm_scratch_bytes(0, M, N, K, synth.DTYPE_BF16)
    assert nbytes > 0
    ws = torch.zeros(nbytes + 16, dtype=torch.uint8, device="cuda")
    out = [torch.empty((M, N), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    print("gemm unaligned workspace", flush=True)
    bm.gemm(0, synth.DTYPE_BF16, M, N, K, A, K, B, K, out[0], N)
    bm.gemm(0, synth.DTYPE_BF16, M, N, K, A, K, B, K, out[1], N, None, ws[4:], nbytes)
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1]) and not ws.any()
