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
                                        (1, 1, [512] * 16, 256), (2, 1, [500] * 16 + [193], 256),
                                        # a weight gradient of one slice, whole and not
                                        (1, 1, [64], 256), (4, 1, [40, 23], 256),
                                        # more than 8 column tiles: four row tiles side by side
                                        (3, 2, [333, 467], 1288)],
                         ids=lambda v: str(v) if isinstance(v, int) else "%d_rows" % sum(v))
def test_row_tiles(E, k, lens, F):
    cfg = moe.moe_cfg(synth.DTYPE_BF16, 512, 4, 2, 128, F, E, k, 0.2)
    moe.test_bf16_choice_is_admissible_and_everything_matches_under_it("moe_tiles", cfg, lens, 71)


def test_infinity_beside_rows_that_fill_up_an_expert():
    """The first token of an expert has an infinite gradient: the rows that fill up the expert's last block read that token's row and
    add nothing, so the expert's weight gradients are infinite where the token reaches and never NaN."""
    import torch
    from paper_2605_25451_amd.runner import CaseOnDevice
    E, d, F, hit = 3, 512, 256, 5
    dev = CaseOnDevice(synth.make_case(moe.moe_cfg(synth.DTYPE_BF16, d, 4, 2, 128, F, E, 2, 0.2), [333, 167], 72, name="moe_inf"))
    dev.forward()
    chosen, _ = dev.moe_routing()
    rows = [int((chosen == e).sum()) for e in range(E)]
    mine = [int(e) for e in chosen[0]]                          # the token in front of theirs
    assert all(rows[e] % 128 for e in mine)
    dev.dy[0, hit] = float("inf")
    print("infinite gradient", rows, flush=True)
    dev.backward()
    torch.cuda.synchronize()
    down, up = dev.runner.grads["w_down"].view(E, d, F), dev.runner.grads["w_up"].view(E, 2 * F, d)
    reached = torch.zeros(d, 1, dtype=torch.bool, device="cuda")
    reached[hit] = True
    for e in range(E):
        assert torch.equal(torch.isinf(down[e]), (reached if e in mine else reached & False).expand(d, F)), e
        assert not torch.isnan(down[e]).any() and not torch.isnan(up[e]).any(), e
        assert bool(torch.isinf(up[e]).all()) == (e in mine) and bool(torch.isfinite(up[e]).all()) == (e not in mine), e
