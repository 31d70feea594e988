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


# sizes that choose it: one round of wide tiles to three of small ones (Q|K|V with rotated heads of 64 and 128, 144 tiles), gate and up
# with more rounds of small ones, beside projections that keep the small tiles
@pytest.mark.parametrize("heads,kv,q,E,S", [(32, 16, 9, 1, 128), (16, 8, 9, 1, 128), (32, 16, 9, 1, 96)])
def test_chosen_tiles_have_the_bits_of_the_small_ones(heads, kv, q, E, S):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="int8", n_layers=1, d_model=2048, n_heads=heads, n_kv_heads=kv, d_ffn=5632, vocab=600, max_seq=256,
                   act="swiglu", norm="rmsnorm", pos="rope", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=16,
                   lora_targets=("q", "v"), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1, eps=1e-2, weight_quant="int8")
    T, dh = 2 * q * E * S, 2048 // heads
    assert M.mpz_debug_gemm_tile(T, 4096, 2048, False, 8, 3072, dh) == (6 if T > 2048 else 12 if dh == 64 else 15)
    assert M.mpz_debug_gemm_tile(T, 5632, 2048, True, 8) == 6 and M.mpz_debug_gemm_tile(T, 2048, 2048, False, 8) != 6
    frozen = W.make_frozen_weights(w, 1)
    masters = W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    hs = []
    for cfg in (0, 12, 1):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_tile_config(m.handle, cfg)
        m.regen_noise(5, 0)
        hs.append(m.run_layers(m.embed(tokens), 0, 1, E, S).clone())
    assert torch.equal(hs[0], hs[1]) and torch.equal(hs[0], hs[2])
