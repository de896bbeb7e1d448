"""Attention kernels with 256 rows per workgroup (needs a GPU).  dK/dV at head size 128: pairs of wavefronts whose
keys end inside, at the edge of and before their 64, query tiles that are cut, fewer query tiles than ring
buffers, grouped heads that are split over workgroups, and more than 64 sequences.  Alternating groups: wavefronts
past the sequence, fewer key tiles than ring slots, one key, and the diagonal in every wavefront.  Each case asserts
the kernels it is for."""
import pytest

import test_gpu_ops as ops
from paper_2605_25451_amd import binding as bm
from paper_2605_25451_amd import synth

pytestmark = pytest.mark.gpu


def check(Hq, Hkv, dh, lens, causal, plan):
    got = bm.probe_attention_plan(causal, Hq, Hkv, dh, synth.cu_from_lengths(lens))
    assert all(want in (None, rows) for want, rows in zip(plan, got)), got
    ops.test_attention_matches_definition(synth.DTYPE_BF16, Hq, Hkv, dh, lens, causal)


RAGGED = [1, 64, 65, 225, 480, 511, 720, 1537, 1280, 1025]


@pytest.mark.parametrize("Hq,Hkv,lens,causal", [
    # three workgroups per CU or more
    (64, 64, [256] * 12, 1), (64, 64, [241, 256, 512, 500, 250, 225, 255, 481, 768, 33, 1], 0),
    (64, 64, [241, 256, 512, 500, 250, 225, 255, 481, 768, 33, 1], 1),
    (32, 8, [1, 65, 225, 511, 720, 1537, 1793, 1025], 0),          # heads of a group split four ways
    # one round where 128 keys per workgroup take two
    (24, 24, [400] * 4, 0), (16, 16, [256] * 9, 0),
    # no table of sequences
    (12, 12, [255 + i % 3 for i in range(66)], 1),
])
def test_attention(Hq, Hkv, lens, causal):
    check(Hq, Hkv, 128, lens, causal, (None, None, 256))


@pytest.mark.parametrize("Hq,Hkv,dh,lens,causal", [
    (32, 32, 64, RAGGED, 0), (32, 8, 64, RAGGED, 0), (8, 8, 64, [4000] + [236 + i % 21 for i in range(66)], 0),
    (24, 24, 128, RAGGED, 0), (24, 8, 128, [1, 64, 193, 225, 511, 720, 1537, 2049, 1280], 1),
    (24, 24, 128, [1793, 1, 1536, 33, 769, 1312], 1),
])
def test_alternating_groups(Hq, Hkv, dh, lens, causal):
    check(Hq, Hkv, dh, lens, causal, (256, 256 if dh == 128 else None, None))


@pytest.mark.parametrize("Hq,Hkv,dh,lens,causal", [
    # packs that were handed to the 256-row kernels and are faster without
    (24, 24, 128, [256, 193, 449, 512, 1], 1), (64, 64, 64, [225, 256, 480, 511, 512, 720, 768, 193, 1], 1),
    (16, 16, 128, [2048, 100, 900, 40], 1), (32, 8, 128, [640] * 4, 1),
])
def test_packs_of_128_rows(Hq, Hkv, dh, lens, causal):
    check(Hq, Hkv, dh, lens, causal, (128, 128, 128))
