"""Norm backward at the widths where its kernels change (needs a GPU): the column sums of the wavefronts that
share or split a row, up to the widest rows, with fewer rows than wavefronts and with a ragged last trip."""
import numpy as np
import pytest

from oracle import block_oracle as bo
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu

VIT, LLM = synth.vit_large, synth.decoder_8b_gqa


@pytest.mark.parametrize("base,head_dim,hidden,lens", [
    (VIT, 64, 512, [3]), (VIT, 64, 1024, [5, 2, 70]), (VIT, 64, 1536, [33]), (VIT, 64, 2048, [9, 4]),
    (VIT, 64, 4096, [6, 1]), (VIT, 64, 8192, [3, 2]),
    (LLM, 128, 1024, [7]), (LLM, 128, 1536, [130]), (LLM, 128, 4096, [1]), (LLM, 128, 8192, [5]),
])
def test_block_gradients(base, head_dim, hidden, lens):
    from paper_2605_25451_amd.runner import CaseOnDevice
    cfg = synth.scaled(base(), hidden=hidden, n_q_heads=hidden // head_dim, n_kv_heads=1, head_dim=head_dim, mlp_hidden=256)
    case = synth.make_case(cfg, lens, hidden + len(lens), name=f"norm_{hidden}")
    dev = CaseOnDevice(case)
    print(f"norm hidden={hidden} lens={lens}", flush=True)
    dev.step()
    y, dx, grads, _ = dev.results()
    ry, rdx, rgrads, _ = bo.block_fwd_bwd(case.cfg, case.params, case.x, case.cu_seqlens, case.dy)
    for name, got, ref in [("y", y, ry), ("dx", dx, rdx)] + [(k, grads[k], rgrads[k]) for k in rgrads]:
        assert np.abs(got - ref).max() <= 2e-2 * np.abs(ref).max(), name     # the bf16 tolerance of the block tests
