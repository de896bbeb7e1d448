"""Attention backward whose dK/dV and dQ tiles share a launch (needs a GPU), on both sides of each line of the rule:
head counts that leave the two-heads workgroup half empty, packs of one workgroup, below a round, between one and one and a
half, and whose dQ fits beside a second round, packs that take two launches, and keys packed on their own, against
attention in float64.  The plan of each case is asserted."""
import numpy as np
import pytest

from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, head size, causal, query lengths, key lengths (None: the queries'), (launches, workgroups of dK/dV, of dQ)
    (1, 1, 128, 0, [1], None, (1, 1, 1)), (3, 1, 128, 1, [130, 5], None, (1, 9, 6)), (3, 3, 72, 0, [129, 64], None, (1, 9, 6)),
    (5, 5, 72, 1, [200], None, (1, 10, 6)),
    (15, 5, 128, 0, [130], None, (1, 30, 16)),                                # odd heads, split over q-head parts
    (8, 8, 128, 0, [700, 650], None, (1, 96, 48)), (8, 8, 128, 1, [1300, 900], None, (1, 152, 76)),    # below a round
    (24, 24, 128, 1, [1100], None, (1, 216, 108)),                            # one to one and a half rounds, causal
    (24, 24, 128, 0, [1100], None, (2, 216, 216)),                            # ... and without a mask
    (12, 12, 128, 0, [1300, 1300], None, (1, 144, 132)),                      # wide dK/dV, a round and a quarter
    (9, 9, 128, 0, [2000, 2300], None, (2, 153, 306)),                        # ... beyond
    (24, 24, 128, 1, [1300], None, (1, 264, 132)),                            # dK/dV beyond a round, dQ in its gaps
    (13, 13, 72, 0, [1300, 1300], None, (1, 286, 154)),                       # ... with an odd number of heads
    (32, 32, 128, 1, [1700], None, (2, 448, 448)), (8, 8, 128, 0, [1300, 1400], None, (2, 176, 176)),
    (24, 24, 72, 0, [400] * 4, None, (2, 384, 384)),
    (32, 8, 128, 1, [4096], None, (1, 1024, 512)),                            # dQ with turns
    (2, 2, 64, 0, [300, 1], None, (1, 8, 8)), (4, 2, 64, 1, [257, 128], None, (1, 16, 16)),
    (4, 4, 128, 0, [100, 200], [0, 333], (1, 12, 6)), (3, 3, 64, 0, [64, 100], [130, 0], (1, 6, 6)),
    (3, 3, 72, 0, [70, 1], [5, 300], (1, 12, 4)),
]


@pytest.mark.parametrize("Hq,Hkv,dh,causal,lq,lk,plan", CASES)
def test_joint_attention_backward(Hq, Hkv, dh, causal, lq, lk, plan):
    import torch
    from paper_2605_25451_amd import binding as bm
    gen = torch.Generator(device="cuda").manual_seed(Hq * 1000 + dh + sum(lq))
    own_keys, lk = lk is not None, lq if lk is None else lk
    cuq, cuk = (np.concatenate([[0], np.cumsum(l)]).astype(np.int32) for l in (lq, lk))
    assert bm.probe_attention_backward_plan(causal, Hq, Hkv, dh, cuq, cuk if own_keys else None) == plan
    Tq, Tk, S = int(cuq[-1]), int(cuk[-1]), len(lq)
    rnd = lambda t, h: torch.randn((t, h * dh), device="cuda", generator=gen).bfloat16()
    q, k, v, d_o = rnd(Tq, Hq), rnd(Tk, Hkv), rnd(Tk, Hkv), rnd(Tq, Hq)
    o, lse = torch.empty_like(q), torch.empty((Hq, Tq), device="cuda")
    dq, dk, dv = (torch.full_like(t, float("nan")) for t in (q, k, v))
    dev = lambda c: torch.from_numpy(c).cuda()
    nbytes = bm.cp_attention_backward_scratch_bytes(Hq, Hkv, dh, Tq, Tk)
    ws = torch.empty(max(nbytes, 16), dtype=torch.uint8, device="cuda")
    print(f"joint attention {Hq}/{Hkv} x {dh} causal={causal} {lq} {lk}", flush=True)
    bm.cp_attention_forward(synth.DTYPE_BF16, causal, Hq, Hkv, dh, q, Hq * dh, k, v, Hkv * dh, dev(cuq), cuq, dev(cuk), cuk, S, o, lse)
    bm.cp_attention_backward(synth.DTYPE_BF16, causal, Hq, Hkv, dh, q, Hq * dh, k, v, Hkv * dh, o, d_o, lse, dev(cuq), cuq, dev(cuk),
                             cuk, S, dq, Hq * dh, dk, dv, Hkv * dh, ws, nbytes)
    torch.cuda.synchronize()
    # float64 on the same inputs, and on the kernel's own rounded o (delta is taken from it)
    h = lambda t: t.cpu().double().view(t.shape[0], -1, dh)
    Q, K, V, O, D = (h(t) for t in (q, k, v, o, d_o))
    rq, rk, rv = torch.zeros_like(Q), torch.zeros_like(K), torch.zeros_like(V)
    for s in range(S):
        a, b = slice(cuq[s], cuq[s + 1]), slice(cuk[s], cuk[s + 1])
        for i in range(Hq):
            j = i // (Hq // Hkv)
            if b.start == b.stop: continue
            sc = Q[a, i] @ K[b, j].T / dh ** 0.5
            if causal: sc = sc.masked_fill(torch.ones_like(sc).triu(1).bool(), float("-inf"))
            p = torch.softmax(sc, -1)
            ds = p * (D[a, i] @ V[b, j].T - (D[a, i] * O[a, i]).sum(-1, keepdim=True)) / dh ** 0.5
            rq[a, i] += ds @ K[b, j]; rk[b, j] += ds.T @ Q[a, i]; rv[b, j] += p.T @ D[a, i]
    for got, ref, name in ((dq, rq, "dq"), (dk, rk, "dk"), (dv, rv, "dv")):
        g = h(got)
        assert torch.isfinite(g).all(), name
        # P and dS are rounded to bf16 in front of their products, the result once more: a few 2^-9 of the largest value
        assert ((g - ref).abs().max() <= 2e-2 * max(ref.abs().max().item(), 1e-30)), name
