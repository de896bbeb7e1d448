"""GELU in the epilogue of the products of few rows (needs a GPU): fp32 rows, columns and bias sums that end inside 16x16 tiles, with
and without biases, at the last rows that it takes and the first where the pass of its own returns, and where only the backward's
does because its bias sums do not fit the workspace, against the oracle.  How many passes of their own a case has is asserted."""
import numpy as np
import pytest

from oracle import block_oracle as bo
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

TINY = synth.vit_tiny()
CASES = {
    "fp32_1": (TINY, [1]), "fp32_16": (TINY, [9, 7]), "fp32_17": (TINY, [17]), "fp32_no_bias": (synth.scaled(TINY, linear_bias=0), [40, 33]),
    "fp32_columns": (synth.scaled(TINY, mlp_hidden=100), [31, 30]), "fp32_300": (TINY, [200, 100]), "fp32_1500": (TINY, [700, 800]),
    "fp32_3008": (TINY, [300] * 10 + [8]), "fp32_3009": (TINY, [300] * 10 + [9]),
    "fp32_sums_fit": (synth.scaled(TINY, mlp_hidden=64), [256] * 16), "fp32_sums_do_not_fit": (synth.scaled(TINY, mlp_hidden=64), [256] * 16 + [1]),
}
PASSES = {"fp32_3009": 2, "fp32_sums_do_not_fit": 1}     # of GELU and its backward; else 0


@pytest.mark.parametrize("name", CASES)
def test_against_oracle(name):
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import CaseOnDevice
    cfg, lens = CASES[name]
    case = synth.make_case(cfg, lens, 23, name=name)
    dev = CaseOnDevice(case)
    print("gelu epilogue", name, flush=True)
    bm.profile_begin()
    dev.step()
    # besides: the column sums of the QKV bias and the fold of all of them
    assert bm.profile_end()["elementwise"][2] == PASSES.get(name, 0) + 1 + cfg.linear_bias
    y, dx, grads, _ = dev.results()
    ref = bo.block_fwd_bwd(case.cfg, case.params, case.x, case.cu_seqlens, case.dy)
    tol = 1e-5                                      # the fp32 block tests' tolerance
    rel = lambda a, b: float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))
    assert rel(y, ref[0]) <= tol and rel(dx, ref[1]) <= tol
    for k, g in ref[2].items():
        assert rel(grads[k], g) <= tol, k
