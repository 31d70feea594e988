"""Causal attention at the edges of its tiles, pieces and blocks (32 queries of a wave, pieces of 64 or 32 keys, blocks of 128 or 256 queries, one
to several pieces, scores kept or computed twice) against the same rounding steps in plain PyTorch: scores and sums in fp32, P rounded
to bf16 against the exact row maximum."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,dh,sizes", [(4, 2, 64, (2, 31, 33, 64, 65, 127, 128, 129, 191, 192, 255, 256, 257, 448, 512)),
                                            (3, 3, 128, (2, 32, 33, 63, 64, 65, 97, 128, 129, 256, 300)), (4, 1, 128, (64, 96))])
def test_every_piece(H, Hkv, dh, sizes):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="att", n_layers=1, d_model=H * dh, n_heads=H, n_kv_heads=Hkv, d_ffn=64, vocab=100, max_seq=512, act="relu", norm="layernorm",
                   pos="learned", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=4, lora_targets=("q",),
                   loss_mode="next_token_all_pos", q=1, E=1, S=32, steps=1, eps=1e-3)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2))
    for S in sizes:
        n = 3
        g = torch.Generator(device="cuda").manual_seed(S)
        x = torch.randn(n * S, (H + 2 * Hkv) * dh, device="cuda", generator=g).bfloat16()
        out = torch.full((n * S + 1, H * dh), 7.0, device="cuda", dtype=torch.bfloat16)
        M.mpz_debug_attention(m.handle, x.data_ptr(), n, S, out.data_ptr())
        assert bool((out[n * S] == 7.0).all())
        q, k, v = x.view(n, S, -1).float().split([H * dh, Hkv * dh, Hkv * dh], -1)
        q = q.reshape(n, S, H, dh).transpose(1, 2)
        k, v = (t.reshape(n, S, Hkv, dh).repeat_interleave(H // Hkv, 2).transpose(1, 2).contiguous() for t in (k, v))
        s = (q @ k.transpose(2, 3).contiguous()) * dh ** -0.5
        s = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
        p = torch.exp(s - s.max(-1, keepdim=True).values).bfloat16().float()
        y = ((p @ v) / p.sum(-1, keepdim=True)).transpose(1, 2).reshape(n * S, H * dh)
        got = out[:n * S].float()
        # a probability that rounds the other way (exp2 against exp, another order of the scores' sums) moves an element by 2^-8 of one of
        # its terms; the output's own rounding is half an ulp
        assert float((got - y).norm() / y.norm()) < 3e-3, S
        assert float((got - y).abs().max()) < 2.0 ** -7 * float(y.abs().max()), S
