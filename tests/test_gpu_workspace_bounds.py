"""Blocks stay inside the workspaces that they ask for (needs a GPU): what lies behind `saved` and `scratch` is untouched by a
step, for every kind of block and for rows that take shared and separate launches."""
import pytest

from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

GUARD = 1 << 20
MOE = synth.scaled(synth.decoder_moe(), hidden=256, n_q_heads=2, n_kv_heads=1, mlp_hidden=128, n_experts=8, top_k=2)
BLOCKS = {
    "tiny_fp32": (synth.vit_tiny(), [40, 33]), "vit": (synth.vit_large(), [300, 277]), "vit_no_bias": (synth.scaled(synth.vit_large(), linear_bias=0), [65]),
    "vit_rope": (synth.scaled(synth.vit_large(), hidden=512, n_q_heads=8, n_kv_heads=8, mlp_hidden=1024, rope=1), [1500]),
    "decoder": (synth.scaled(synth.decoder_7b(), hidden=384, n_q_heads=3, n_kv_heads=3, mlp_hidden=1536), [1000, 301]),
    "gqa": (synth.scaled(synth.decoder_8b_gqa(), hidden=1024, n_q_heads=8, n_kv_heads=2, mlp_hidden=2048), [777]),
    "dit": (synth.scaled(synth.dit_block(), hidden=576, n_q_heads=8, n_kv_heads=8, mlp_hidden=1152), [100] * 9), "moe": (MOE, [200, 57]),
}


def guarded(nbytes):
    import torch
    t = torch.full((nbytes + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    return t, t[nbytes:]


def check(dev, holder):
    import torch
    dev.saved, behind_saved = guarded(holder.saved_bytes)
    holder.scratch, behind_scratch = guarded(holder.scratch_bytes)
    dev.step()
    dev.step()
    torch.cuda.synchronize()
    assert bool((behind_saved == 0xA5).all()), "saved"
    assert bool((behind_scratch == 0xA5).all()), "scratch"


@pytest.mark.parametrize("kind", BLOCKS)
def test_block(kind):
    from paper_2605_25451_amd.runner import CaseOnDevice
    cfg, lens = BLOCKS[kind]
    dev = CaseOnDevice(synth.make_case(cfg, lens, 3, name=kind))
    print("block", kind, flush=True)
    check(dev, dev.runner)


def test_two_stream_block():
    from paper_2605_25451_amd.runner import TwoStreamOnDevice
    cfg = synth.scaled(synth.dit_block(), hidden=512, n_q_heads=4, n_kv_heads=4, head_dim=128, mlp_hidden=1024)
    dev = TwoStreamOnDevice(synth.make_two_stream_case(cfg, [33, 129], [300, 64], 71, 1, "two_stream"))
    print("two-stream block", flush=True)
    check(dev, dev)
