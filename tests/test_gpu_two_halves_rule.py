"""Which passes run as two halves on two streams: the tokens and widths on either side of the rule, with the bits of the pass on one stream."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,q,E,S,streams,quant", [(16, 8, 2, 96, 1, "none"),      # 1024 wide, 3072 tokens: one pass fills its rounds as well
                                                 (16, 9, 2, 128, 2, "none"),     # 4608
                                                 (16, 16, 1, 144, 2, "none"),    # the same in copies of 144 rows
                                                 (16, 10, 2, 128, 1, "none"),    # 5120
                                                 (12, 8, 2, 170, 1, "none"),     # 768 wide, 5440 tokens: below 3 x 2^30
                                                 (12, 8, 4, 128, 1, "none"),     # 8192
                                                 (12, 8, 4, 136, 2, "none"),     # 8704
                                                 (32, 8, 2, 96, 1, "none"),     # 2048 wide
                                                 (16, 9, 4, 128, 2, "int8"),    # 9216
                                                 (16, 8, 4, 128, 1, "int8")])   # 8192
def test_streams_and_bits(heads, q, E, S, streams, quant):
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="halves", n_layers=1, d_model=64 * heads, n_heads=heads, n_kv_heads=heads if heads == 12 else heads // 2,
                   d_ffn=1024, vocab=600, max_seq=256, act="swiglu", norm="rmsnorm", pos="rope", has_bias=False, tie_embeddings=False,
                   dtype="bf16", lora_rank=8, lora_targets=("q", "v"), loss_mode="last_pos_label_subset", q=q, E=E, S=S, steps=1, eps=1e-2, weight_quant=quant)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05))
    tokens, labels = torch.from_numpy(W.make_tokens(w, 3)).cuda(), torch.from_numpy(W.make_labels(w, 3)).cuda()
    m.regen_noise(5, 0)
    got = m.forward_perturbed(tokens, labels).clone()
    assert M.mpz_debug_last_pass_streams(m.handle) == streams
    M.mpz_debug_set_two_halves(m.handle, False)
    one = m.forward_perturbed(tokens, labels).clone()
    assert M.mpz_debug_last_pass_streams(m.handle) == 1
    assert torch.equal(got.view(torch.int32), one.view(torch.int32))


@pytest.mark.parametrize("quant,q,streams", [("none", 10, 2), ("none", 11, 1), ("int8", 13, 2), ("int8", 8, 1)])
def test_wide_models(quant, q, streams):
    """d = 2560, 256 tokens per query: both wide projections a little over one round of 256-wide tiles (300 and 270; int8 390 and 351)."""
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.Workload(name="halves", n_layers=1, d_model=2560, n_heads=40, n_kv_heads=40, d_ffn=6912, vocab=600, max_seq=128, act="relu",
                   norm="layernorm", pos="learned", has_bias=True, tie_embeddings=True, dtype="bf16", lora_rank=8, lora_targets=("q", "v"),
                   loss_mode="last_pos_label_subset", q=q, E=1, S=128, steps=1, eps=1e-2, weight_quant=quant)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05))
    tokens, labels = torch.from_numpy(W.make_tokens(w, 3)).cuda(), torch.from_numpy(W.make_labels(w, 3)).cuda()
    m.regen_noise(5, 0)
    got = m.forward_perturbed(tokens, labels).clone()
    assert M.mpz_debug_last_pass_streams(m.handle) == streams
    M.mpz_debug_set_two_halves(m.handle, False)
    one = m.forward_perturbed(tokens, labels).clone()
    assert M.mpz_debug_last_pass_streams(m.handle) == 1
    assert torch.equal(got.view(torch.int32), one.view(torch.int32))
