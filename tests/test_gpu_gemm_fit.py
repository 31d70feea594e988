"""The tiles fitted to rounds of CUs (8 waves, operands fetched straight into LDS, persistent blocks) against the register-staged 128 x 128
tile, which sums in the same order: every bit.  Shapes 20 .. 25: 192 x 256, 256 x 192, 192 x 128, 128 x 192, 256 x 128, 128 x 128 (features x
tokens); 26: int8 256 x 256.  Sizes: fewer rows than a tile, ragged rows and columns, K of one, two and three K-tiles (fewer than the stages), more tiles than
blocks (a block then walks two or three, the fetches running on across the epilogue and more than one tile ahead)."""
import pytest

pytestmark = pytest.mark.gpu

FITTED = (20, 21, 22, 23, 24, 25)
SHAPES = [(32, 256, 64), (300, 264, 192), (256, 256, 5504), (4640, 4360, 128), (8224, 2312, 256), (6000, 4616, 64)]


@pytest.mark.parametrize("m,n,k", SHAPES)
@pytest.mark.parametrize("act,f32,bias", [(-1, False, False), (0, False, True), (-1, False, True), (-1, True, True), (2, False, False), (2, False, True)])
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
    for cfg in (1,) + FITTED:
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
        M.mpz_debug_gemm_bf16(m, n, k, x.data_ptr(), w.data_ptr(), None if b is None else b.data_ptr(), act, out.data_ptr(), f32, st, cfg)
        assert bool((out[m] == -7.0).all())               # nothing past the last row
        outs.append(out[:m])
    for cfg, out in zip(FITTED, outs[1:]):
        assert torch.equal(out, outs[0]), cfg


@pytest.mark.parametrize("m,n,k", [(32, 256, 64), (300, 264, 192), (256, 256, 5504), (4640, 4360, 128), (6000, 4616, 64)])
@pytest.mark.parametrize("act,f32,bias", [(-1, False, False), (0, False, True), (-1, True, True), (2, False, False), (2, False, True)])
def test_int8_equals_the_staged_tile(m, n, k, act, f32, bias):
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m * 7 + n + k + act)
    nw = 2 * n if act == 2 else n
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = torch.randint(-127, 128, (nw, k), generator=g, device="cuda", dtype=torch.int8)
    scale = torch.rand(nw, generator=g, device="cuda") * 1e-3 + 1e-4
    b = torch.randn(nw, generator=g, device="cuda") if bias else None
    st = torch.cuda.current_stream().cuda_stream
    outs = []
    for cfg in (1, 21, 23, 24, 25, 26):
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
        M.mpz_debug_gemm_int8(m, n, k, x.data_ptr(), w.data_ptr(), scale.data_ptr(), None if b is None else b.data_ptr(), act, out.data_ptr(),
                              f32, st, cfg)
        assert bool((out[m] == -7.0).all())
        outs.append(out[:m])
    for out in outs[1:]:
        assert torch.equal(out, outs[0])


@pytest.mark.parametrize("quant", ["none", "int8"])
@pytest.mark.parametrize("kind,heads,q,E,S,rank", [("rope64", 8, 4, 1, 64, 8), ("rope64", 8, 2, 3, 96, 16), ("rope128", 4, 2, 2, 64, 16),
                                                   ("rope128", 4, 5, 1, 32, 8), ("plain", 12, 4, 1, 64, 8), ("plain", 12, 3, 1, 160, 16)])
def test_model_pass_with_a_fitted_tile_forced(kind, heads, q, E, S, rank, quant):
    """Two blocks with low-rank terms (rank 8 and 16), rotary embedding, residual and SwiGLU / ReLU epilogues, every bit of the residual
    stream.  Copies of 32 to 288 rows: a wave's tokens span several.  768 wide: segments that the 192-wide tiles take.  Heads of 128 columns: the
fitted tiles rotate them, the staged one (and what stands in for the 192-wide shapes and, bf16, 26, which rotate nothing) leaves that to a kernel
of its own, one launch a block."""
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    llama = kind != "plain"
    w = W.Workload(name="fit", n_layers=2, d_model=heads * (128 if kind == "rope128" else 64), n_heads=heads, n_kv_heads=4 if llama else heads,
                   d_ffn=640, vocab=600, max_seq=256, act="swiglu" if llama else "relu", norm="rmsnorm" if llama else "layernorm",
                   pos="rope" if llama else "learned", has_bias=not llama, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                   lora_targets=("q", "k", "v", "o"), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1, eps=1e-2,
                   weight_quant=quant)
    frozen = W.make_frozen_weights(w, 1)
    masters = W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    hs, rotary = [], []
    for cfg in (1,) + FITTED + (26,):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_tile_config(m.handle, cfg)
        m.regen_noise(5, 0)
        M.mpz_profile_begin(m.handle)
        hs.append(m.run_layers(m.embed(tokens), 0, 2, E, S).clone())
        rotary.append(M.mpz_profile_end(m.handle)["rope"]["launches"])
    if kind == "rope128":
        assert rotary == [2, 2, 0, 2, 0, 0, 0, 0 if quant == "int8" else 2]
    for cfg, h in zip(FITTED + (26,), hs[1:]):
        assert torch.equal(h.view(torch.int32), hs[0].view(torch.int32)), cfg


# the choice by size: 128 x 128 tiles of a round and a half, three part-filled rounds of 256 x 256 ones; gate and up; the edges where the tile
# stays: 128 small tiles, fp32 apart; four rounds of the large one
@pytest.mark.parametrize("m,n,k,dual,tile", [(3072, 2048, 1024, False, 23), (1536, 12288, 4096, False, 23), (2048, 4096, 4096, False, 24),
                                             (1536, 5632, 2048, True, 23), (2176, 1024, 1024, False, 25), (2048, 1024, 1024, False, -1),
                                             (320, 11008, 4096, True, -1), (32768, 4096, 2048, False, -1)])
def test_choice_by_size_has_the_bits_of_the_staged_tile(m, n, k, dual, tile):
    import torch
    import paper_2409_15520_amd as M
    assert M.mpz_debug_gemm_fitted_tile(m, n, k, dual) == tile
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = (torch.randn(2 * n if dual else n, k, generator=g, device="cuda") * 0.05).bfloat16()
    outs = []
    for cfg in (0, 1):
        out = torch.empty(m, n, device="cuda", dtype=torch.bfloat16)
        M.mpz_debug_gemm_bf16(m, n, k, x.data_ptr(), w.data_ptr(), None, 2 if dual else -1, out.data_ptr(), False,
                              torch.cuda.current_stream().cuda_stream, cfg)
        outs.append(out)
    assert torch.equal(outs[0], outs[1])
