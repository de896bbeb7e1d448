"""Input and weight gradients that share a launch (needs a GPU): the gradients of a block whose products meet the rule,
at rows that end inside tiles and slices, with one and with several k ranges, against the oracle; and the sizes where the
rule gives way to separate launches."""
import numpy as np
import pytest

from oracle import block_oracle as bo
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

VIT = dict(hidden=512, n_q_heads=8, n_kv_heads=8, head_dim=64, mlp_hidden=1024)
CASES = [
    # fp32: 16x16 tiles that end inside the rows and columns; 72: past the rows of a tile, 300: more workgroups than CUs
    (synth.vit_tiny(), [1]), (synth.vit_tiny(), [17, 14]), (synth.vit_tiny(), [40, 32]), (synth.vit_tiny(), [200, 100]),
    # bf16: one partial slice of rows, rows that end inside a slice, k ranges on both sides, and few tiles a slot
    (synth.scaled(synth.vit_large(), **VIT), [40]), (synth.scaled(synth.vit_large(), **VIT), [65, 64]),
    (synth.scaled(synth.vit_large(), **VIT), [130, 127, 256]), (synth.scaled(synth.vit_large(), **VIT), [513, 300]),
    (synth.scaled(synth.dit_block(), hidden=576, n_q_heads=8, n_kv_heads=8, mlp_hidden=1152), [100, 100, 57]),
    (synth.scaled(synth.decoder_7b(), hidden=512, n_q_heads=4, n_kv_heads=4, mlp_hidden=1024), [129, 70]),
]


@pytest.mark.parametrize("cfg,lens", CASES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, list) else "d%d" % v.hidden)
def test_joint_gradients(cfg, lens):
    from paper_2605_25451_amd.runner import CaseOnDevice
    case = synth.make_case(cfg, lens, 11, name="joint")
    dev = CaseOnDevice(case)
    print(f"joint gradients hidden={cfg.hidden} rows={sum(lens)}", flush=True)
    dev.step()
    dev.step()                                      # accumulates: the weight gradients double
    y, dx, grads, dcond = dev.results()
    ref = bo.block_fwd_bwd(case.cfg, case.params, case.x, case.cu_seqlens, case.dy,
                           **({} if case.cond is None else {"cond": case.cond}))
    tol = 1e-5 if cfg.dtype == synth.DTYPE_FP32 else 2e-2        # the block tests' tolerances: storage type, chained roundings
    rel = lambda a, b: float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))
    assert rel(dx, ref[1]) <= tol
    for k, g in ref[2].items():
        assert rel(grads[k], 2.0 * g) <= tol, k
