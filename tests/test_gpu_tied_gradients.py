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


VIT_256 = synth.scaled(synth.vit_large(), hidden=256, n_q_heads=4, n_kv_heads=4, mlp_hidden=512)


@pytest.mark.parametrize("lens,ranges", [([500, 268], 3), ([156, 100], 1)], ids=["3_ranges", "1_range"])
def test_tied_qkv_and_output_weights_add_up(lens, ranges):
    """The weight gradients of the QKV and output projections share a launch; with accumulators that overlap, here the last
    rows of w_qkv's and the first ones of w_o's, they have one each."""
    import torch
    from paper_2605_25451_amd import binding as bm
    from paper_2605_25451_amd.runner import CaseOnDevice
    assert bm.probe_block_weight_gradients(bm.make_desc(VIT_256), sum(lens), len(lens)) == (0, 0, ranges, ranges)
    dev = CaseOnDevice(synth.make_case(VIT_256, lens, 5, name="tied_qkv_o"))
    run = dev.runner

    def weight_gradient_launches():             # alone or with each other: one beside an input gradient counts as that
        bm.profile_begin()
        dev.step()
        _, flops, count = bm.profile_end()["gemm_tn"]
        torch.cuda.synchronize()
        return count, flops
    print("separate accumulators", flush=True)
    apart = weight_gradient_launches()
    g = {k: v.clone() for k, v in run.grads.items()}
    d, qkv = VIT_256.hidden, VIT_256.qkv_dim
    both = torch.zeros(qkv + d // 2, d, device="cuda")
    run.g = bm.make_params(dict(run.grads, w_qkv=both[:qkv], w_o=both[qkv - d // 2:]))
    run.zero_grads()
    print("tied accumulators", flush=True)
    assert weight_gradient_launches() != apart
    want = torch.zeros_like(both)
    want[:qkv] += g["w_qkv"]
    want[qkv - d // 2:] += g["w_o"]
    # the same products with their k ranges cut elsewhere: 2-norm error of an fp32 sum over 768 rows, 2^-24 * sqrt(768) = 1.7e-6
    assert float((both - want).norm() / want.norm()) <= 1e-5
    for k in ("w_up", "w_down", "b_qkv", "b_o"):
        assert torch.equal(run.grads[k], g[k]), k
