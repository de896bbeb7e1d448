"""Gain and bias gradients that share one accumulator (tied parameters) are added one after the other (needs a GPU):
the folded column sums of a backward pass run in one launch only where their accumulators are distinct."""
import pytest

from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg,lens", [(synth.vit_tiny(), [17, 23]), (synth.scaled(synth.vit_large(), mlp_hidden=1024), [130, 65])],
                         ids=["fp32", "bf16"])
def test_tied_gradients_add_up(cfg, lens):
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import CaseOnDevice
    dev = CaseOnDevice(synth.make_case(cfg, lens, 5, name="tied"))
    run = dev.runner
    print("separate accumulators", flush=True)
    dev.step()
    torch.cuda.synchronize()
    g = {k: v.clone() for k, v in run.grads.items()}
    # the second pair overlaps in part: b_o starts half way into b_down's accumulator
    d = cfg.hidden
    gain, biases = torch.zeros(d, device="cuda"), torch.zeros(d + d // 2, device="cuda")
    tied = dict(run.grads, norm1_g=gain, norm2_g=gain, b_down=biases[:d], b_o=biases[d // 2:])
    run.g = bm.make_params(tied)
    run.zero_grads()
    print("tied accumulators", flush=True)
    dev.step()
    torch.cuda.synchronize()
    # one fp32 addition of the same two sums: exact
    assert torch.equal(gain, g["norm2_g"] + g["norm1_g"])
    want = torch.zeros_like(biases)
    want[:d] += g["b_down"]
    want[d // 2:] += g["b_o"]
    assert torch.equal(biases, want)
    for k in ("norm1_b", "norm2_b", "b_up", "b_qkv"):
        assert torch.equal(run.grads[k], g[k]), k
