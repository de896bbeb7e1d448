"""Mixture-of-experts block at widths around the two gathers (needs a GPU): a thread per 16 bytes, and a wavefront per
row that fills one or two trips or leaves the last of four part empty, against the oracle on the fp32 path."""
import pytest

import test_gpu_moe as moe
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,seed", [(24, 63), (128, 60), (256, 60), (264, 60), (512, 60), (520, 60), (776, 60)])
def test_widths(hidden, seed):
    cfg = moe.moe_cfg(synth.DTYPE_FP32, hidden, hidden // 8, hidden // 8, 8, 32, 6, 2, 0.3)
    moe.test_fp32_check_path_matches_oracle("moe_d%d" % hidden, cfg, [17, 40, 5, 1], seed)
