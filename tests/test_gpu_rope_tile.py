"""The 128 x 128 tile with four waves of 128 x 32 rotates heads of 128 columns in its epilogue (what mid-size passes of 7B-shaped
models take): every bit of the 64 x 64-wave tile followed by the rotary kernel, bf16 and int8 weights, rank 8 and 16, segments on
some and on all of Q, K and V, a last token tile of 64 rows and one of 32."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("quant", ["none", "int8"])
@pytest.mark.parametrize("q,E,S,rank,targets,kv", [(1, 5, 32, 16, "qkvo", 4), (2, 1, 96, 8, "qv", 2), (1, 1, 32, 16, "k", 4), (3, 1, 160, 8, "qkvo", 1)])
def test_fused_heads_of_128(quant, q, E, S, rank, targets, kv):
    import torch
    import paper_2409_15520_amd as M
    w = W.Workload(name="rope128", n_layers=2, d_model=512, n_heads=4, n_kv_heads=kv, d_ffn=640, vocab=600, max_seq=256, act="swiglu",
                   norm="rmsnorm", pos="rope", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=tuple(targets), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1, eps=1e-2, weight_quant=quant)
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    outs, rotary = [], []
    for cfg in (15, 1):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_tile_config(m.handle, cfg)
        m.regen_noise(5, 0)
        M.mpz_profile_begin(m.handle)
        outs.append(m.run_layers(m.embed(tokens), 0, 2, E, S).clone())
        rotary.append(M.mpz_profile_end(m.handle)["rope"]["launches"])
    assert rotary == [0, 2]                                # fused in one, a kernel of its own per block in the other
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1])
