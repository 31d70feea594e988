"""The LoRA bottleneck of few tokens (a block per 32 tokens and target, LDS ring): the same bits as the kernel of many
tokens, at every rank it takes, against a batch too large for it.  (Copies of 33 and 45 rows, and rank 12, take kernels of their
own whatever the batch: the same comparison for those.)"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


# one block's worth of sequences alone (few blocks) and repeated until a block per CU is exceeded; K = 1024 (four chunks, as many
# as stages) and 2048
@pytest.mark.parametrize("rank,d,S", [(8, 1024, 32), (16, 1024, 33), (32, 1024, 64), (16, 2048, 45), (12, 1024, 32),
                                      (16, 1024, 32), (16, 2048, 64), (8, 2048, 32)])
def test_few_tokens_equal_many(rank, d, S):
    import torch
    import paper_2409_15520_amd as M
    many = 8192 // S + 1                                   # copies x sequences x tokens past 256 blocks for any number of targets
    w = W.Workload(name="few", n_layers=1, d_model=d, n_heads=d // 64, n_kv_heads=d // 64, d_ffn=256, vocab=500, max_seq=64,
                   act="relu", norm="layernorm", pos="learned", has_bias=True, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=("o",), loss_mode="next_token_all_pos", q=1, E=many, S=S, steps=1, eps=1e-2)
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    outs = []
    for E in (1, many):
        m = M.ZoModel(w.with_(E=E), frozen, masters)
        M.mpz_debug_set_split_k(m.handle, False)           # one summation order whatever the number of rows
        m.regen_noise(5, 0)
        tok = tokens[:E].contiguous()
        h = m.run_layers(m.embed(tok), 0, 1, E, S).reshape(2, E, S, -1)
        outs.append(h[:, 0].clone())
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("rank,S", [(16, 32), (8, 64)])
def test_rows_that_begin_between_pieces(rank, S):
    """Operand rows that begin on 8 bytes but not on 16 keep the kernels that fetch through registers: the same bits."""
    import torch
    import paper_2409_15520_amd as M
    w = W.Workload(name="shift", n_layers=1, d_model=1024, n_heads=16, n_kv_heads=16, d_ffn=256, vocab=500, max_seq=64, act="relu",
                   norm="layernorm", pos="learned", has_bias=True, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=("q", "v"), loss_mode="next_token_all_pos", q=1, E=1, S=S, steps=1, eps=1e-2)
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05))
    m.regen_noise(5, 0)
    T = 2 * S
    x = torch.randn(T * 1024 + 4, generator=torch.Generator(device="cuda").manual_seed(rank), device="cuda").bfloat16()
    outs = []
    for buf in (x[4:], x[4:].clone()):
        out = torch.empty(T, 3072, device="cuda")
        M.mpz_debug_qkv_projection(m.handle, buf.data_ptr(), 0, 1, S, out.data_ptr())
        outs.append(out)
    assert x[4:].data_ptr() % 16 == 8 and torch.equal(outs[0], outs[1])
