"""Attention kernels with 256 rows per workgroup (needs a GPU).  dK/dV at head size 128: pairs of wavefronts whose
keys end inside, at the edge of and before their 64, query tiles that are cut, fewer query tiles than ring
buffers, grouped heads that are split over workgroups, and more than 64 sequences.  Alternating groups: wavefronts
past the sequence, fewer key tiles than ring slots, one key, and the diagonal in every wavefront."""
import pytest

import test_gpu_ops as ops
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,lens,causal", [
    # three workgroups per CU or more
    (64, 64, [256] * 12, 1), (64, 64, [241, 256, 512, 500, 250, 225, 255, 481, 768, 33, 1], 0),
    (64, 64, [241, 256, 512, 500, 250, 225, 255, 481, 768, 33, 1], 1), (32, 8, [1000, 770, 255, 512, 2048, 1501], 1),
    # one round where 128 keys per workgroup take two
    (24, 24, [400] * 4, 0), (24, 24, [256, 193, 449, 512, 1], 1), (16, 16, [256] * 9, 0),
    # no table of sequences
    (12, 12, [255 + i % 3 for i in range(66)], 1),
])
def test_attention(Hq, Hkv, lens, causal):
    ops.test_attention_matches_definition(synth.DTYPE_BF16, Hq, Hkv, 128, lens, causal)


@pytest.mark.parametrize("Hq,Hkv,dh,lens,causal", [
    (64, 64, 64, [256] * 9, 1), (64, 16, 64, [1, 64, 65, 224, 225, 256, 480, 511, 512, 720, 768], 0),
    (64, 64, 64, [225, 256, 480, 511, 512, 720, 768, 193, 1], 1), (32, 32, 64, [250 + i for i in range(66)], 0),
    (64, 64, 128, [225, 256, 480, 511, 512, 720, 768, 64, 33], 0), (64, 32, 128, [225, 256, 480, 511, 512, 720, 768, 193, 1], 1),
])
def test_alternating_groups(Hq, Hkv, dh, lens, causal):
    ops.test_attention_matches_definition(synth.DTYPE_BF16, Hq, Hkv, dh, lens, causal)
