"""Attention of a sequence whose rows span more than 4 GiB: keys and values past what the offsets into one buffer reach, at queries all over the
sequence, against plain PyTorch in fp32 with P rounded to bf16 against the exact maximum."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,dh,S", [(128, 64, 87489), (64, 128, 87501)])
def test_rows_past_four_gib(H, dh, S):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    d = H * dh
    w = W.Workload(name="far", n_layers=1, d_model=d, n_heads=H, n_kv_heads=H, d_ffn=64, vocab=100, max_seq=64, act="relu", norm="layernorm",
                   pos="learned", has_bias=False, tie_embeddings=False, dtype="bf16", lora_rank=4, lora_targets=("q",),
                   loss_mode="next_token_all_pos", q=1, E=1, S=32, steps=1, eps=1e-3)
    m = M.ZoModel(w, M.device_random_weights(w, 1), W.make_lora_masters(w, 2))
    assert S * 3 * d * 2 > (1 << 32) + 64 * 6 * d
    g = torch.Generator(device="cuda").manual_seed(S)
    x = torch.empty(S, 3 * d, device="cuda", dtype=torch.bfloat16)
    for r in range(0, S, 8192):
        x[r:r + 8192] = torch.randn(min(8192, S - r), 3 * d, device="cuda", generator=g)
    x[:, :d] *= 2.0                                        # scores far enough apart that a row of zeros for a key shows
    out = torch.full((S + 1, d), 7.0, device="cuda", dtype=torch.bfloat16)
    M.mpz_debug_attention(m.handle, x.data_ptr(), 1, S, out.data_ptr())
    assert bool((out[S] == 7.0).all())
    rows = torch.tensor([0, 31, 64, 127, S // 3, S // 2 - 1, S // 2, S * 3 // 4, S - 65, S - 2, S - 1], device="cuda")
    q = x[rows, :d].float().view(-1, H, dh).transpose(0, 1).contiguous()
    for head in (0, H // 2, H - 1):
        k, v = (x[:, o + head * dh:o + (head + 1) * dh].float() for o in (d, 2 * d))
        s = (q[head] @ k.t().contiguous()) * dh ** -0.5
        s = s.masked_fill(torch.arange(S, device="cuda")[None] > rows[:, None], float("-inf"))
        p = torch.exp(s - s.max(-1, keepdim=True).values).bfloat16().float()
        y = (p @ v) / p.sum(-1, keepdim=True)
        got = out[rows, head * dh:(head + 1) * dh].float()
        # the bounds of test_gpu_attention_pieces: a probability that rounds the other way moves an element by 2^-8 of one of its terms
        assert float((got - y).norm() / y.norm()) < 3e-3, head
        assert float((got - y).abs().max()) < 2.0 ** -7 * float(y.abs().max()), head
