"""The large GEMM tile (operands fetched straight into LDS, persistent blocks) against the register-staged tiles, which sum in
the same order: every bit.  Sizes: fewer rows than a tile, ragged rows and columns, the smallest K, more tiles than blocks (a
block then walks several tiles, the operand fetches running on across the epilogue), with 1 / 2 / 43 K-tile pairs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(32, 256, 128), (300, 264, 256), (256, 256, 5504), (4640, 4360, 128), (8224, 2312, 256)]


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("act,f32,bias", [(-1, False, False), (0, False, True), (0, False, False), (-1, False, True), (-1, True, True),
                                          (-1, True, False), (2, False, False), (2, False, True)])
def test_equals_the_staged_tile(m, n, k, act, f32, bias):
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m * 7 + n + k + act)
    nw = 2 * n if act == 2 else n
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = (torch.randn(nw, k, generator=g, device="cuda") * 0.05).bfloat16()
    b = torch.randn(nw, generator=g, device="cuda") if bias else None
    st = torch.cuda.current_stream().cuda_stream
    outs = []
    for cfg in (6, 1):
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
        M.mpz_debug_gemm_bf16(m, n, k, x.data_ptr(), w.data_ptr(), None if b is None else b.data_ptr(), act, out.data_ptr(), f32,
                              st, cfg)
        assert bool((out[m] == -7.0).all())               # nothing past the last row
        outs.append(out[:m])
    assert torch.equal(outs[0], outs[1])
    # and both are the product: fp32 sums of K bf16 products against 64 bits, plus the output's own rounding
    y = x.double() @ w.double().t()
    if b is not None:
        y = y + b.double()
    if act == 2:
        y = torch.nn.functional.silu(y[:, :n]) * y[:, n:]
    elif act == 0:
        y = torch.relu(y)
    err = float((outs[0].double() - y).norm() / y.norm())
    assert err < (2e-6 if f32 else 2.0 ** -8)             # fp32: sqrt(K) 2^-24 ~ 5e-6 at worst x rms of partial sums; bf16: half an ulp


@pytest.mark.parametrize("cfg_shape", [("rope64", 4, 1, 64, 8), ("rope64", 2, 3, 96, 16), ("rope128", 2, 2, 64, 16), ("plain", 4, 1, 64, 8),
                                       ("plain", 3, 1, 160, 16)])
def test_model_pass_with_the_large_tile_forced(cfg_shape):
    """A block with low-rank terms (rank 8 and 16), rotary embedding, residual and SwiGLU / ReLU epilogues: the large tile
    forced against the 128-wide one, every bit of the residual stream.  Copies of 64 to 288 rows: a tile spans several."""
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    kind, q, E, S, rank = cfg_shape
    llama = kind != "plain"
    w = W.Workload(name="pipe", n_layers=2, d_model=512, n_heads=4 if kind == "rope128" else 8, n_kv_heads=4, d_ffn=640, vocab=600,
                   max_seq=256, act="swiglu" if llama else "relu", norm="rmsnorm" if llama else "layernorm",
                   pos="rope" if llama else "learned", has_bias=not llama, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=("q", "k", "v", "o") if llama else ("q", "v"), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1,
                   eps=1e-2)
    frozen = W.make_frozen_weights(w, 1)
    masters = W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    hs, ls = [], []
    for cfg in (6, 1):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_tile_config(m.handle, cfg)
        m.regen_noise(5, 0)
        h = m.run_layers(m.embed(tokens), 0, 2, E, S)
        hs.append(h.clone())
        ls.append(m.head_loss(h, tokens).cpu().numpy().astype(np.float64))
    assert torch.equal(hs[0], hs[1])
    # the fused cross-entropy folds other column groups: fp32 exponentials and sums of 600 terms
    assert np.abs(ls[0] - ls[1]).max() / ls[1].max() < 1e-6
