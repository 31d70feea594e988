"""fp32 models on the 64-bit matrix instructions: parity with the oracle at the edges of the tiles (16 x 16 and 32 x 32, K by
quarters of 16), with K that no quarter divides and sequences of up to 129 tokens.  Both sides
sum in binary64 and round every stored value once, so only values next to a rounding border may differ: the bar of the
other fp32 parity tests."""
import numpy as np
import pytest

from gpu_helpers import gpu_steps, make_bundle, oracle_steps, rel_err
from small_workloads import MICRO, MINI_LLAMA, MINI_OPT

pytestmark = pytest.mark.gpu

SHAPES = {
    "d36_heads_of_6": MINI_LLAMA.with_(d_model=36, n_heads=6, n_kv_heads=3, d_ffn=52, q=1, E=1, S=15, max_seq=16, lora_rank=4),
    "d20_ffn_17_general": MINI_OPT.with_(d_model=20, n_heads=2, n_kv_heads=2, d_ffn=17, q=1, E=1, S=10, lora_rank=8),
    "S128_big_tiles": MINI_OPT.with_(d_model=64, n_heads=4, n_kv_heads=4, d_ffn=260, q=2, E=2, S=128, max_seq=129, lora_rank=12),
    "S129": MICRO.with_(q=1, E=1, S=129, max_seq=129, lora_rank=4),
    "S17_heads_of_64": MINI_LLAMA.with_(d_model=128, n_heads=2, n_kv_heads=1, d_ffn=96, q=2, E=3, S=17, max_seq=32, lora_rank=64,
                                        lora_targets=("q", "o")),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_fp32_shapes(name):
    b = make_bundle(SHAPES[name], b_std=0.02)
    Lg, Gg, Mg = gpu_steps(b, 1)
    Lo, Go, Mo = oracle_steps(b, 1)
    assert np.abs(Lg - Lo).max() <= 1e-6 * np.abs(Lo).max()
    assert rel_err(Gg[0], Go[0]) <= 1e-4
    assert rel_err(Mg, Mo) <= 1e-3


def test_bottleneck_of_more_waves_than_a_launch_holds():
    """Rank 64 on Q, K and V from 1.4 M stacked tokens on: 2^32 threads at a wave per row and four columns.  A sequence's rows do not
    depend on how many others there are."""
    import torch
    import paper_2409_15520_amd as M
    import workloads as W
    big = 5500
    w = W.Workload(name="wide", n_layers=1, d_model=32, n_heads=2, n_kv_heads=2, d_ffn=32, vocab=64, max_seq=128, act="relu",
                   norm="layernorm", pos="learned", has_bias=True, tie_embeddings=True, dtype="f32", lora_rank=64,
                   lora_targets=("q", "k", "v"), loss_mode="next_token_all_pos", q=1, E=big, S=128, steps=1, eps=1e-2)
    assert 2 * big * 128 * 3 * 64 // 4 * 64 >= 2 ** 32
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    outs = []
    for first, E in ((0, big), (0, 3), (big - 3, 3)):
        m = M.ZoModel(w.with_(E=E), frozen, masters)
        m.regen_noise(5, 0)
        outs.append(m.run_layers(m.embed(tokens[first:first + E].contiguous()), 0, 1, E, 128).reshape(2, E, 128, -1).clone())
        m.close()
    assert torch.equal(outs[0][:, :3], outs[1]) and torch.equal(outs[0][:, -3:], outs[2])


def test_embedding_of_the_largest_batch():
    """2^24 stacked tokens, the most a handle takes."""
    import torch
    import paper_2409_15520_amd as M
    import workloads as W
    w = W.Workload(name="most", n_layers=1, d_model=4, n_heads=1, n_kv_heads=1, d_ffn=4, vocab=64, max_seq=512, act="relu",
                   norm="layernorm", pos="learned", has_bias=True, tie_embeddings=True, dtype="f32", lora_rank=4,
                   lora_targets=("q",), loss_mode="last_pos_label_subset", q=1, E=1 << 14, S=512, steps=1, eps=1e-2)
    frozen = W.make_frozen_weights(w, 1)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    m = M.ZoModel(w, frozen, W.make_lora_masters(w, 2))
    m.regen_noise(5, 0)
    h = m.embed(tokens).reshape(2, w.E, w.S, 4)
    want = torch.from_numpy(frozen["emb"]).cuda()[tokens.long()] + torch.from_numpy(frozen["pos_emb"]).cuda()[None, :w.S]
    assert torch.equal(h[0], want) and torch.equal(h[1], want)
