"""Input and weight gradients that share a launch (needs a GPU): the gradients of a block whose products meet the rule,
at rows that end inside tiles and slices and at whole ones, with one and with several k ranges on either side, and where
the rule gives way to separate launches, against the oracle.  The plan of each case is asserted."""
import numpy as np
import pytest

from oracle import block_oracle as bo
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

VIT = dict(hidden=512, n_q_heads=8, n_kv_heads=8, head_dim=64, mlp_hidden=1024)
VIT_256 = synth.scaled(synth.vit_large(), hidden=256, n_q_heads=4, n_kv_heads=4, mlp_hidden=512)
DECODER_256 = synth.scaled(synth.decoder_7b(), hidden=256, n_q_heads=2, n_kv_heads=2, mlp_hidden=1024)
APART = (0, 0)
CASES = [
    # config, lengths, (k ranges of the input gradient, of the weight gradient) of the three pairs
    # fp32: 16x16 tiles that end inside the rows and columns; 72: past the rows of a tile, 300: more workgroups than CUs
    (synth.vit_tiny(), [1], [(1, 1)] * 3), (synth.vit_tiny(), [17, 14], [(1, 1)] * 3), (synth.vit_tiny(), [40, 32], [(1, 1)] * 3),
    (synth.vit_tiny(), [200, 100], [(1, 1)] * 3),
    # bf16: one partial slice of rows, rows that end inside a slice, and few tiles a slot
    (synth.scaled(synth.vit_large(), **VIT), [40], [(4, 1), (1, 1), (6, 1)]),
    (synth.scaled(synth.vit_large(), **VIT), [65, 64], [(4, 1), (1, 1), (6, 1)]),
    (synth.scaled(synth.vit_large(), **VIT), [130, 127, 256], [(1, 1), (1, 1), (2, 1)]),
    (synth.scaled(synth.vit_large(), **VIT), [513, 300], [(1, 1), (1, 3), (1, 1)]),
    (synth.scaled(synth.dit_block(), hidden=576, n_q_heads=8, n_kv_heads=8, mlp_hidden=1152), [100, 100, 57], [(3, 1), (1, 1), (4, 1)]),
    (synth.scaled(synth.decoder_7b(), hidden=512, n_q_heads=4, n_kv_heads=4, mlp_hidden=1024), [129, 70], [(7, 1), (1, 1), (5, 1)]),
    # k ranges on both sides: the partial tiles of the weight gradient lie behind those of the input gradient
    (synth.scaled(synth.decoder_7b(), hidden=384, n_q_heads=3, n_kv_heads=3, mlp_hidden=1536), [1000, 301], [(3, 2), (1, 3), (1, 2)]),
    # rows that are whole slices: the kernels without a cut, with and without ranges on either side
    (VIT_256, [40, 24], [(1, 1)] * 3), (VIT_256, [500, 268], [(1, 1), (1, 3), APART]), (DECODER_256, [64], [(8, 1), (1, 1), (1, 1)]),
    (DECODER_256, [596, 300], [(4, 2), (1, 3), APART]),
    # pairs that are launched apart: few tiles for the slices of the other, many tiles
    (VIT_256, [156, 100], [(1, 1), (1, 1), APART]),
    (synth.scaled(synth.decoder_7b(), hidden=1024, n_q_heads=8, n_kv_heads=8, mlp_hidden=4096), [40], [(16, 1), APART, (12, 1)]),
]


@pytest.mark.parametrize("cfg,lens,plan", CASES, ids=["d%d-%s" % (c.hidden, "-".join(map(str, n))) for c, n, _ in CASES])
def test_joint_gradients(cfg, lens, plan):
    from paper_2605_25451_amd.runner import CaseOnDevice
    from paper_2605_25451_amd import binding as bm
    assert bm.probe_block_backward_plan(bm.make_desc(cfg), sum(lens), len(lens)) == plan
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
