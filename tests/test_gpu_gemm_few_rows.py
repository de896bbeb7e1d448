"""Partial tiles and weight gradients whose wavefronts have no row, one strip of 16 rows or more of a tile to store
(needs a GPU), on 128x128 tiles with one and with several k ranges."""
import pytest

import test_gpu_gemm_tiles as tiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout,M,N,K,split", [
    (layout, M, 264, 4104, True) for layout in (0, 1) for M in (1, 15, 16, 17, 64, 65, 80, 81, 128, 145)
] + [(2, M, N, K, split) for M, N in ((64, 72), (72, 72), (80, 200), (88, 136), (144, 64), (208, 80)) for K, split in ((200, False), (4001, True))])
def test_rows_of_the_last_tile(layout, M, N, K, split):
    tiles.test_gemm_tiles(layout, M, N, K, tiles.T128, split, True)
