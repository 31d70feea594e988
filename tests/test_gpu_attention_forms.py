"""Forms of the attention kernel that have the same bits.  All keys in half the ring: the form that keeps its scores (few sequences) and the one
that computes them twice (heads of 128 that share no keys, more than the last-level cache holds; heads of 64 keep them in any batch).  Four waves
a block (few blocks) and eight; packed batches in eight waves, whose sequences end inside a block or before it."""
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


@pytest.mark.parametrize("H,Hkv", [(4, 2), (4, 4)])
@pytest.mark.parametrize("S,n", [(192, 40), (193, 33), (224, 40), (255, 64), (256, 40), (448, 20), (449, 17), (511, 20), (512, 32)])
def test_eight_waves_have_the_bits_of_four(H, Hkv, S, n):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="att", n_layers=1, d_model=H * 64, n_heads=H, n_kv_heads=Hkv, d_ffn=64, vocab=100, max_seq=512, act="relu", norm="layernorm",
                   pos="learned", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=4, lora_targets=("q",),
                   loss_mode="next_token_all_pos", q=1, E=1, S=32, steps=1, eps=1e-3)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2))
    x = torch.randn(n * S, (H + 2 * Hkv) * 64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(S)).bfloat16()
    all_ = torch.full((n * S + 1, H * 64), 7.0, device="cuda", dtype=torch.bfloat16)
    M.mpz_debug_attention(m.handle, x.data_ptr(), n, S, all_.data_ptr())
    assert bool((all_[n * S] == 7.0).all())
    for s in range(0, n, 8):                                # at most 64 blocks of eight waves: four waves
        k = min(8, n - s)
        few = torch.empty(k * S, H * 64, device="cuda", dtype=torch.bfloat16)
        M.mpz_debug_attention(m.handle, x[s * S:].data_ptr(), k, S, few.data_ptr())
        assert torch.equal(few, all_[s * S:(s + k) * S])


@pytest.mark.parametrize("S,q,lengths", [(256, 4, (256, 2, 33, 192, 129)), (224, 5, (31, 224, 128, 65)), (512, 2, (512, 256, 40, 300, 257)), (480, 2, (2, 480, 448, 225, 255))])
def test_packed_batches_in_eight_waves(S, q, lengths):
    """Against the right-padded batch of 64 more columns, whose attention takes four waves."""
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    E = len(lengths)
    assert 128 < 2 * q * E * 4 * -(-S // 256) <= 256 and (S + 63) % 256 < 191
    w = W.Workload(name="packed8", n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, d_ffn=512, vocab=600, max_seq=S + 64, act="swiglu", norm="rmsnorm",
                   pos="rope", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=8, lora_targets=("q", "v"),
                   loss_mode="next_token_all_pos", q=q, E=E, S=S + 64, steps=1, eps=1e-2)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05))
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    lens = torch.tensor(lengths, dtype=torch.int32, device="cuda")
    m.regen_noise(5, 0)
    padded = m.forward_perturbed(tokens, None, lens).clone()
    packed = m.forward_perturbed_packed(tokens[:, :S].contiguous(), None, lens).clone()
    assert torch.isfinite(packed).all() and len(set(packed.tolist())) == 2 * q
    assert float((packed - padded).abs().max()) <= 1e-6 * float(padded.abs().max())
