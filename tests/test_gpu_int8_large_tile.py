"""int8 weights on the 256-wide tile, which mid-size passes of wide models take: every bit of the 128-wide tiles, with rotated heads
of 64 and 128, low-rank terms, residual, gate and up, copies that end inside a tile."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,q,E,S,rank", [(8, 4, 1, 64, 8), (8, 2, 3, 96, 16), (4, 2, 2, 64, 16)])
def test_block_has_the_bits_of_the_small_tiles(heads, q, E, S, rank):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="int8", n_layers=1, d_model=512, n_heads=heads, n_kv_heads=heads // 2, d_ffn=640, vocab=600, max_seq=256,
                   act="swiglu", norm="rmsnorm", pos="rope", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=("q", "k", "v", "o"), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1, eps=1e-2,
                   weight_quant="int8")
    frozen = W.make_frozen_weights(w, 1)
    masters = W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    hs = []
    for cfg in (6, 1, 12):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_tile_config(m.handle, cfg)
        m.regen_noise(5, 0)
        hs.append(m.run_layers(m.embed(tokens), 0, 1, E, S).clone())
    assert torch.equal(hs[0], hs[1]) and torch.equal(hs[0], hs[2])
