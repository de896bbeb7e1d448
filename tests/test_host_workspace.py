"""Workspaces hold what a block can use (no GPU): nothing for column sums without biases, for per-sequence sums without
adaLN, for the token map without positions; and they grow with the tokens."""
import pytest

from paper_2605_25451_amd import binding as bm
from paper_2605_25451_amd import synth

MB = 1 << 20


def sizes(cfg, T, S=1):
    return bm.block_sizes(bm.make_desc(cfg), T, S, T)


def up256(n):
    return (n + 255) // 256 * 256


@pytest.mark.parametrize("T", [40, 777, 8192])
def test_saved_holds_no_token_map_without_positions(T):
    c = synth.vit_large()
    parts = [8 * T, 8 * T, 4 * c.n_q_heads * T, 2 * T * c.qkv_dim, 2 * T * c.hidden, 2 * T * c.hidden, 2 * T * c.up_dim]
    assert sizes(c, T)[0] == sum(map(up256, parts))
    assert sizes(synth.scaled(c, rope=1), T)[0] == sum(map(up256, parts)) + up256(4 * T)


def test_column_sums_only_for_biases():
    c = synth.vit_large()
    with_bias, without = (sizes(synth.scaled(c, linear_bias=b), 8192)[1] for b in (1, 0))
    assert with_bias - without >= 2 * MB * 2          # up and qkv, about 2 MB each


@pytest.mark.parametrize("cfg,T", [(synth.decoder_7b(), 8192), (synth.decoder_8b_gqa(), 32768)])
def test_scratch_is_the_activations_and_little_more(cfg, T):
    """Beside the gradients of the activations and attention's workspace: 64 MB of partial products, 32 MB of partial rows
    of the norms (with column sums that nothing writes it was 228 MB)."""
    d = cfg.hidden
    rows = 2 * (2 * cfg.mlp_hidden + cfg.up_dim + 3 * d + cfg.n_q_heads * cfg.head_dim + cfg.qkv_dim)
    known = rows * T + bm.attention_backward_scratch_bytes(cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim, T)
    assert sizes(cfg, T)[1] <= known + 100 * MB


@pytest.mark.parametrize("cfg", [synth.vit_tiny(), synth.vit_large(), synth.decoder_7b(), synth.dit_block(), synth.decoder_moe()],
                         ids=["tiny", "vit", "decoder", "dit", "moe"])
def test_scratch_grows_with_tokens(cfg):
    got = [sizes(cfg, T)[1] for T in range(1, 3000, 7)]
    assert got == sorted(got)
