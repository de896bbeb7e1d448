"""Attention backward whose gradients take the place of inputs (needs a GPU): no tile reads what another one of the same
launch has overwritten, so the results are those of buffers of their own, bit for bit."""
import numpy as np
import pytest

from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

BF16, FP32 = synth.DTYPE_BF16, synth.DTYPE_FP32
PACKS = [
    # dtype, Hq, Hkv, head size, causal, lengths
    (BF16, 4, 4, 64, 0, [700, 513]), (BF16, 4, 2, 64, 1, [700, 513]),
    (BF16, 3, 3, 72, 0, [300, 129]),                                      # two heads side by side
    (BF16, 8, 8, 128, 0, [700, 650]), (BF16, 8, 2, 128, 1, [700, 650]),
    (BF16, 24, 24, 128, 0, [1152] * 4), (BF16, 32, 8, 128, 1, [4096]),    # turns, wide and narrow dK/dV
    (FP32, 4, 4, 16, 0, [300, 40]), (FP32, 4, 2, 64, 1, [200, 100]),
]


def places(dtype, Hq, Hkv):
    out = [{"dq": "o"}]
    if Hq == Hkv:
        out.append({"dk": "o"})
    return out + ([{"dq": "q"}, {"dq": "d_o"}] if dtype == BF16 else [{"dk": "k", "dv": "v"}])


@pytest.mark.parametrize("dtype,Hq,Hkv,dh,causal,lens", PACKS)
def test_gradients_in_the_place_of_inputs(dtype, Hq, Hkv, dh, causal, lens):
    import torch
    from paper_2605_25451_amd import binding as bm
    gen = torch.Generator(device="cuda").manual_seed(dh + sum(lens))
    cu = synth.cu_from_lengths(lens)
    T, S, cu_dev = int(cu[-1]), len(lens), torch.from_numpy(cu).cuda()
    rnd = lambda h: torch.randn((T, h * dh), device="cuda", generator=gen).to(torch.bfloat16 if dtype == BF16 else torch.float32)
    given = {"q": rnd(Hq), "k": rnd(Hkv), "v": rnd(Hkv), "d_o": rnd(Hq), "o": rnd(Hq)}
    lse = torch.empty((Hq, T), device="cuda")
    nbytes = bm.cp_attention_backward_scratch_bytes(Hq, Hkv, dh, T, T)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    bm.cp_attention_forward(dtype, causal, Hq, Hkv, dh, given["q"], Hq * dh, given["k"], given["v"], Hkv * dh, cu_dev, cu, cu_dev, cu, S,
                            given["o"], lse)

    def backward(place):
        t = {k: v.clone() for k, v in given.items()}
        g = {"dq": torch.empty_like(t["q"]), "dk": torch.empty_like(t["k"]), "dv": torch.empty_like(t["v"])}
        g.update((grad, t[inp]) for grad, inp in place.items())
        print(f"attention backward {Hq}/{Hkv} x {dh} causal={causal} {lens} {place}", flush=True)
        bm.cp_attention_backward(dtype, causal, Hq, Hkv, dh, t["q"], Hq * dh, t["k"], t["v"], Hkv * dh, t["o"], t["d_o"], lse, cu_dev, cu,
                                 cu_dev, cu, S, g["dq"], Hq * dh, g["dk"], g["dv"], Hkv * dh, ws, nbytes)
        torch.cuda.synchronize()
        return g
    apart = backward({})
    for place in places(dtype, Hq, Hkv):
        got = backward(place)
        for k in apart:
            assert torch.equal(got[k], apart[k]), (place, k)
