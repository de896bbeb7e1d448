"""Products whose rows lie on tiles of two heights (needs a GPU): whole rounds of 256x256 tiles and the other rows on 128x256, with
rows, columns and contractions that end inside tiles and slices, and every epilogue.  The plan of each case is asserted."""
import pytest

import test_gpu_block as block
import test_gpu_gemm_tiles as gemm
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

TWO_HEIGHTS = (384, 256)


@pytest.mark.parametrize("layout,M,N,K", [(0, 5121, 4496, 328), (0, 6204, 5256, 64), (0, 4300, 5384, 1024), (1, 3874, 3976, 216),
                                          (1, 4300, 4096, 520), (1, 3333, 5384, 1024)])
def test_products(layout, M, N, K):
    gemm.test_gemm_tiles(layout, M, N, K, TWO_HEIGHTS, False, True)


@pytest.mark.parametrize("hidden,mlp,T,product", [
    (512, 2688, 3301, (0, "2F", "d")),          # SwiGLU forward
    (512, 2688, 6203, (1, "F", "d")),           # SwiGLU backward
    (1536, 512, 11003, (0, "d", "F")),          # residual
])
def test_fused_epilogues(hidden, mlp, T, product):
    from paper_2605_25451_amd import binding as bm
    size = {"d": hidden, "F": mlp, "2F": 2 * mlp}
    assert bm.probe_gemm_plan(product[0], T, size[product[1]], size[product[2]], 0)[:2] == TWO_HEIGHTS
    cfg = synth.scaled(synth.decoder_8b_gqa(), hidden=hidden, n_q_heads=hidden // 128, n_kv_heads=1, mlp_hidden=mlp)
    case = synth.make_case(cfg, [500] * (T // 500) + [T % 500], T, name=f"two_heights_{hidden}_{mlp}_{T}")
    block.compare(case, block.run_hip(case), block.run_oracle(case))
