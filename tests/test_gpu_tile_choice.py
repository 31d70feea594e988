"""The tile that a mid-size bf16 pass chooses: the bits of the forced 128 x 128 tiles where 192-wide tiles end in a part column, where gate and
up take the 256-wide tile from half a round, where whole 128 x 128 tiles replace halves, and where 64 x 64 ones replace the ring."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,ffn,q,E,S,rank,targets,what,tile", [
    (40, 2816, 4, 2, 128, 16, "qv", "o", 11),              # 192-wide tiles, 64 of 192 features in the last
    (16, 5632, 4, 1, 96, 16, "qvo", "up", 6),              # gate and up: 132 tiles
    (32, 5632, 5, 1, 109, 8, "qv", "o", 12),               # 144 whole tiles, the last rows a part
    (32, 4096, 3, 1, 48, 16, "qkvo", "down", 10)])         # 576 tiles of 32 x 32: 64 x 64 ones
def test_block_has_the_bits_of_whole_tiles(heads, ffn, q, E, S, rank, targets, what, tile):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    d, T = 64 * heads, 2 * q * E * S
    assert M.mpz_debug_gemm_tile(T, *{"o": (d, d), "up": (ffn, d), "down": (d, ffn)}[what], what == "up") == tile
    w = W.Workload(name="mid", n_layers=1, d_model=64 * heads, n_heads=heads, n_kv_heads=heads // 2, d_ffn=ffn, vocab=600, max_seq=256,
                   act="swiglu", norm="rmsnorm", pos="rope", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=tuple(targets), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1, eps=1e-2)
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


# 2304 columns of which 2176 are rotated: by the 128-wide tiles, where the wide one would be chosen without a rotation
@pytest.mark.parametrize("heads,kv,quant", [(32, 2, "none"), (32, 2, "int8"), (16, 1, "none"), (16, 1, "int8")])
def test_rotated_columns_that_end_inside_a_wide_tile(heads, kv, quant):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    bits, dh = 8 if quant == "int8" else 16, 2048 // heads
    assert M.mpz_debug_gemm_tile(10240, 2304, 2048, False, bits) == 6
    assert M.mpz_debug_gemm_tile(10240, 2304, 2048, False, bits, 2176, dh) == (15 if dh == 128 else 12)
    w = W.Workload(name="mid", n_layers=1, d_model=2048, n_heads=heads, n_kv_heads=kv, d_ffn=256, vocab=600, max_seq=256, act="swiglu",
                   norm="rmsnorm", pos="rope", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=16, lora_targets=("q",),
                   loss_mode="next_token_all_pos", q=10, E=2, S=256, steps=1, eps=1e-2, weight_quant=quant)
    frozen = W.make_frozen_weights(w, 1)
    masters = W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    hs = []
    for cfg in (0, 12, 1):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_tile_config(m.handle, cfg)
        m.regen_noise(5, 0)
        hs.append(m.run_layers(m.embed(tokens), 0, 1, 2, 256).clone())
    assert torch.equal(hs[0], hs[1]) and torch.equal(hs[0], hs[2])
