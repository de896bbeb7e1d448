"""Which launches the backward of the GPU tests' cases takes (no GPU): a line of a rule that moves past a case shows here."""
import numpy as np
import pytest

import test_gpu_joint_attention as attention
import test_gpu_joint_gradients as gradients
import test_gpu_weight_gradients as weights
from paper_2605_25451_amd import binding as bm
from paper_2605_25451_amd import synth


@pytest.mark.parametrize("Hq,Hkv,dh,causal,lq,lk,plan", attention.CASES)
def test_attention(Hq, Hkv, dh, causal, lq, lk, plan):
    cuq, cuk = (None if l is None else np.concatenate([[0], np.cumsum(l)]).astype(np.int32) for l in (lq, lk))
    assert bm.probe_attention_backward_plan(causal, Hq, Hkv, dh, cuq, cuk) == plan


@pytest.mark.parametrize("cfg,lens,plan", gradients.CASES)
def test_gradients(cfg, lens, plan):
    assert bm.probe_block_backward_plan(bm.make_desc(cfg), sum(lens), len(lens)) == plan


def test_every_variant_of_the_joint_products_has_a_case():
    """(input gradient split, weight gradient split, rows end inside a slice)"""
    seen = {(a > 1, b > 1, sum(lens) % 64 != 0) for cfg, lens, plan in gradients.CASES if cfg.dtype == synth.DTYPE_BF16
            for a, b in plan if (a, b) != gradients.APART}
    assert len(seen) == 8


def test_full_packs_share_no_launch_with_an_input_gradient():
    assert bm.probe_block_backward_plan(bm.make_desc(synth.vit_large()), 16384, 28) == [(0, 0)] * 3
    assert bm.probe_block_backward_plan(bm.make_desc(synth.decoder_7b()), 8192, 8) == [(0, 0)] * 3


@pytest.mark.parametrize("cfg,T,ranges", [
    (synth.vit_large(), 16384, (1, 1, 1, 1)), (synth.decoder_7b(), 8192, (1, 1, 1, 1)), (synth.dit_block(), 16384, (1, 1, 8, 1)),
    (synth.scaled(synth.vit_large(), hidden=512, n_q_heads=8, n_kv_heads=8, mlp_hidden=2048), 16384, (5, 5, 5, 5)),
    # past 16384 rows the QKV and output projection alone, or none; fewer than 1024 rows beside input gradients
    (synth.vit_large(), 20000, (0, 0, 4, 4)), (synth.decoder_8b_gqa(), 32768, (0, 0, 0, 0)), (synth.decoder_7b(), 777, (0, 0, 0, 0)),
    (synth.vit_tiny(), 40, (0, 0, 0, 0))])
def test_weight_gradients_of_a_pack(cfg, T, ranges):
    assert bm.probe_block_weight_gradients(bm.make_desc(cfg), T, 1) == ranges


def test_weight_gradient_cases():
    for name, (cfg, lens) in weights.CASES.items():
        assert bm.probe_block_weight_gradients(bm.make_desc(cfg), sum(lens), len(lens)) == weights.RANGES[name], name


@pytest.mark.parametrize("layout,M,N,K", [(0, 3301, 5376, 64), (0, 2566, 13424, 200), (1, 4631, 11600, 176), (0, 5430, 3000, 304),
                                          (1, 2186, 8552, 448), (1, 1469, 12288, 128), (0, 8205, 4096, 224), (1, 4429, 4096, 320)])
def test_short_and_ragged_products_keep_the_smallest_tile(layout, M, N, K):
    """Tiles of two heights give way to the 128x128 tile under six slices and where the columns end inside a cache line."""
    assert bm.probe_gemm_plan(layout, M, N, K) == (128, 128, 1)


@pytest.mark.parametrize("layout,M,N,K", [(0, 2238, 9216, 400), (1, 5376, 4096, 376), (0, 3301, 5376, 512)])
def test_whole_lines_of_columns_take_two_heights(layout, M, N, K):
    assert bm.probe_gemm_plan(layout, M, N, K) == (384, 256, 1)


def test_bad_arguments():
    desc = bm.make_desc(synth.vit_large())
    for T, S in ((0, 1), (4, 5), (4, 0)):
        with pytest.raises(bm.BmError):
            bm.probe_block_backward_plan(desc, T, S)
        with pytest.raises(bm.BmError):
            bm.probe_block_weight_gradients(desc, T, S)
        with pytest.raises(bm.BmError):
            bm.probe_mmdit_weight_gradients(bm.make_mmdit_desc(synth.dit_block(), 1), T, 8, S)
    with pytest.raises(bm.BmError):
        bm.probe_block_backward_plan(bm.make_desc(synth.decoder_moe()), 64, 1)
    with pytest.raises(bm.BmError):
        bm.probe_block_weight_gradients(bm.make_desc(synth.decoder_moe()), 64, 1)
    with pytest.raises(bm.BmError):
        bm.probe_attention_backward_plan(2, 4, 4, 64, [0, 8])
    assert bm.probe_attention_backward_plan(0, 4, 4, 16, [0, 8]) == (0, 0, 0)
