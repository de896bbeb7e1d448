"""All weight gradients of a block in one launch at the end of its backward (needs a GPU): rows that end inside slices and
tiles and whole ones, with one k range each, with all of them split and with one that is, against the oracle; accumulators
that share memory.  The k ranges of each case are asserted."""
import numpy as np
import pytest

from oracle import block_oracle as bo
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

VIT = synth.vit_large()
CASES = {
    # 8 tiles, all split; 1111 rows end inside a slice, 8000 are whole slices
    "all_split": (synth.scaled(VIT, hidden=256, n_q_heads=4, n_kv_heads=4, mlp_hidden=512), [600, 511]),
    "all_split_whole": (synth.scaled(VIT, hidden=256, n_q_heads=4, n_kv_heads=4, mlp_hidden=512), [1000] * 8),
    # tiles that end inside the columns, no bias, SwiGLU
    "ragged_columns": (synth.scaled(synth.decoder_7b(), hidden=384, n_q_heads=3, n_kv_heads=3, mlp_hidden=1160), [1500, 1273]),
    # 192 tiles, one range each
    "one_range": (VIT, [577, 900, 523]),
    "one_range_whole": (VIT, [1024] * 3),
    # 275 tiles with a gate in front of the output projection, whose gradient is split over a round of its own
    "one_split": (synth.dit_block(), [256] * 15 + [250]),
}
# of the down, up, output and QKV projection
RANGES = {"all_split": (4, 4, 4, 4), "all_split_whole": (14, 14, 14, 14), "ragged_columns": (4, 4, 4, 4), "one_range": (1, 1, 1, 1),
          "one_range_whole": (1, 1, 1, 1), "one_split": (1, 1, 6, 1)}
rel = lambda a, b: float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-30))


@pytest.mark.parametrize("name", CASES)
def test_against_oracle(name):
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import CaseOnDevice
    cfg, lens = CASES[name]
    assert bm.probe_block_backward_plan(bm.make_desc(cfg), sum(lens), len(lens)) == [(0, 0)] * 3
    assert bm.probe_block_weight_gradients(bm.make_desc(cfg), sum(lens), len(lens)) == RANGES[name]
    case = synth.make_case(cfg, lens, 19, name=name)
    dev = CaseOnDevice(case)
    print("weight gradients", name, flush=True)
    dev.step()
    dev.step()                                      # accumulates: the weight gradients double
    y, dx, grads, dcond = dev.results()
    ref = bo.block_fwd_bwd(case.cfg, case.params, case.x, case.cu_seqlens, case.dy,
                           **({} if case.cond is None else {"cond": case.cond}))
    assert rel(dx, ref[1]) <= 2e-2                  # the block tests' tolerance: bf16 storage, chained roundings
    for k, g in ref[2].items():
        assert rel(grads[k], 2.0 * g) <= 2e-2, k


def test_tied_accumulators_add_up():
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import CaseOnDevice
    cfg, lens = CASES["all_split"]
    dev = CaseOnDevice(synth.make_case(cfg, lens, 5, name="tied"))
    run = dev.runner
    dev.step()
    torch.cuda.synchronize()
    g = {k: v.clone() for k, v in run.grads.items()}
    both = torch.zeros(cfg.mlp_hidden * cfg.hidden, device="cuda")
    run.g = bm.make_params(dict(run.grads, w_up=both.view(cfg.mlp_hidden, cfg.hidden), w_down=both.view(cfg.hidden, cfg.mlp_hidden)))
    run.zero_grads()
    print("tied accumulators", flush=True)
    dev.step()
    torch.cuda.synchronize()
    # the same products with their k ranges cut elsewhere: 2-norm error of an fp32 sum over 1111 rows, 2^-24 * sqrt(1111) = 2e-6
    want = g["w_up"].flatten() + g["w_down"].flatten()
    assert float((both - want).norm() / want.norm()) <= 1e-5
    for k in ("w_o", "w_qkv"):
        assert float((run.grads[k] - g[k]).norm() / g[k].norm()) <= 1e-5, k


TWO_STREAMS = [
    # lengths of either stream, k ranges of either
    ([500, 800], [1100, 900], ((1, 1, 1, 0), (1, 1, 1, 1))), ([40, 33], [1000, 1111], ((0, 0, 0, 0), (1, 1, 1, 1))),
    ([1024, 1024], [70, 9], ((2, 2, 2, 0), (0, 0, 0, 0))),
]


@pytest.mark.parametrize("text,image,ranges", TWO_STREAMS, ids=["both", "image", "text"])
def test_two_stream_block(text, image, ranges):
    """Streams long enough for a shared launch, both and either of them, with rows that end inside tiles and whole ones."""
    import test_gpu_mmdit as mmdit
    from paper_2605_25451_amd import binding as bm
    cfg = synth.scaled(synth.dit_block(), hidden=1024, n_q_heads=8, n_kv_heads=8, head_dim=128, mlp_hidden=2048)
    assert bm.probe_mmdit_weight_gradients(bm.make_mmdit_desc(cfg, 1), sum(text), sum(image), len(text)) == ranges
    case = synth.make_two_stream_case(cfg, text, image, 75, 1, "two_stream_weights")
    print("two-stream weight gradients", flush=True)
    mmdit.compare(case, mmdit.run_hip(case), mmdit.run_oracle(case))


def test_bias_sums_of_more_sequences_than_fit():
    """The sums of the gated gradients beside the gates: a row per part of a sequence; more of them than the workspace has go a
    way of their own."""
    from paper_2605_25451_amd.runner import CaseOnDevice
    case = synth.make_case(synth.dit_block(), [1] * 900 + [3] * 40, 29, name="many")
    dev = CaseOnDevice(case)
    dev.step()
    y, dx, grads, dcond = dev.results()
    ref = bo.block_fwd_bwd(case.cfg, case.params, case.x, case.cu_seqlens, case.dy, cond=case.cond)
    assert rel(dx, ref[1]) <= 2e-2
    for k, g in ref[2].items():
        assert rel(grads[k], g) <= 2e-2, k
