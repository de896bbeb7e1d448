"""Experts whose rows fill one, two and three row blocks, exactly and with a remainder (needs a GPU): two blocks share a 256-row
tile and the last one of an odd number has a tile of its own; widths that end inside a tile and k ranges that end inside a slice; rows
that are read by their token and rows that are sorted first."""
import pytest

import test_gpu_moe as moe
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k,lens,F", [(1, 1, [128], 256), (1, 1, [129], 256), (1, 1, [256], 264), (1, 1, [200, 57], 256),
                                        (1, 1, [300, 340], 136), (3, 2, [333, 167], 256), (4, 1, [260, 380], 264),
                                        # the most rows whose tokens a weight gradient looks up itself, and one pack that is sorted first
                                        (1, 1, [512] * 16, 256), (2, 1, [500] * 16 + [193], 256)],
                         ids=lambda v: str(v) if isinstance(v, int) else "%d_rows" % sum(v))
def test_row_tiles(E, k, lens, F):
    cfg = moe.moe_cfg(synth.DTYPE_BF16, 512, 4, 2, 128, F, E, k, 0.2)
    moe.test_bf16_choice_is_admissible_and_everything_matches_under_it("moe_tiles", cfg, lens, 71)
