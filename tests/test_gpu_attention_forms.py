"""Attention of all keys in half the ring: the form that keeps its scores (few sequences) and the one
that computes them twice (heads of 128 that share no keys, more than the last-level cache holds; heads of 64 keep them in any batch)
have the same bits."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Hkv,dh,S,n", [(32, 4, 64, 128, 256), (32, 4, 64, 120, 280), (16, 8, 64, 97, 512), (20, 20, 128, 64, 256), (20, 20, 128, 33, 520)])
def test_both_forms_have_the_same_bits(H, Hkv, dh, S, n):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="att", n_layers=1, d_model=H * dh, n_heads=H, n_kv_heads=Hkv, d_ffn=64, vocab=100, max_seq=128, act="relu", norm="layernorm",
                   pos="learned", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=4, lora_targets=("q",),
                   loss_mode="next_token_all_pos", q=1, E=1, S=32, steps=1, eps=1e-3)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2))
    x = torch.randn(n * S, (H + 2 * Hkv) * dh, device="cuda", generator=torch.Generator(device="cuda").manual_seed(S)).bfloat16()
    all_ = torch.empty(n * S, H * dh, device="cuda", dtype=torch.bfloat16)
    M.mpz_debug_attention(m.handle, x.data_ptr(), n, S, all_.data_ptr())
    step = 40
    for s in range(0, n, step):
        k = min(step, n - s)
        few = torch.empty(k * S, H * dh, device="cuda", dtype=torch.bfloat16)
        M.mpz_debug_attention(m.handle, x[s * S:].data_ptr(), k, S, few.data_ptr())
        assert torch.equal(few, all_[s * S:(s + k) * S])
