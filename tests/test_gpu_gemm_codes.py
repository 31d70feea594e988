"""The streamed few-token GEMM on 4-bit weights: every token tile (64 / 128 / 192 / 256) with ragged tokens, features that end inside
a tile, tiles shared by several blocks and blocks that span tiles, each epilogue of the reduction, against 64-bit products; and a
model's block whose copies differ strongly, against the pass that dequantises its weights."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 33, 64, 65, 128, 129, 192, 193, 256])
@pytest.mark.parametrize("n,k,act,residual", [(4100, 2112, -1, True), (300, 11008, 0, False), (2052, 4096, 2, False), (22016, 1024, -1, False)])
def test_streamed_codes(m, n, k, act, residual):
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    nw = 2 * n if act == 2 else n
    codes = torch.randint(0, 256, (nw, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    absmax = (0.048 * (0.5 + torch.rand(nw, k // 64, device="cuda", generator=g))).contiguous()
    w = torch.empty(nw, k, dtype=torch.bfloat16, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    M.mpz_debug_dequant_nf4(codes.data_ptr(), absmax.data_ptr(), w.data_ptr(), nw * k, st)
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    r = torch.randn(m, n, generator=g, device="cuda") if residual else None
    partial = torch.empty(20 * m * nw, device="cuda")
    outs = []
    for _ in range(2):
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if residual else torch.bfloat16)
        partial.fill_(float("nan"))                        # a slot nobody wrote would show
        M.mpz_debug_gemm_nf4_splitk(m, n, k, x.data_ptr(), codes.data_ptr(), absmax.data_ptr(), None, act,
                                    None if r is None else r.data_ptr(), out.data_ptr(), residual, -1, partial.data_ptr(), partial.numel(), st)
        assert bool((out[m] == -7.0).all())
        outs.append(out[:m])
    assert torch.equal(outs[0], outs[1])
    y = x.double() @ w.double().t()
    if act == 2:
        y = torch.nn.functional.silu(y[:, :n]) * y[:, n:]
    elif act == 0:
        y = torch.relu(y)
    if r is not None:
        y = y + r.double()
    err = float((outs[0].double() - y).norm() / y.norm())
    assert err < (2e-6 if residual else 2.0 ** -8)         # fp32 sums of K products; bf16 rounding of the output


# Q|K|V and gate, up of the 7B shape, whose runs of Q|K|V (16 of 64 K-tiles) end with their tiles; a width of 5632, where a block ends one tile
# (88 K-tiles in runs of 23) and begins the next one with its low-rank term
@pytest.mark.parametrize("q,S,rank,d,run", [(1, 96, 16, 4096, 16), (2, 64, 16, 4096, 16), (4, 32, 8, 4096, 16), (1, 96, 16, 5632, 23), (4, 32, 8, 5632, 23)])
def test_block_with_low_rank_terms(q, S, rank, d, run):
    """192 and 256 tokens of 2 to 8 copies, perturbed by as much as the adapters are large."""
    import torch
    import workloads as W
    import paper_2409_15520_amd as M
    w = W.get_workload("c5_llama7b").with_(n_layers=1, q=q, E=1, S=S, weight_quant="nf4", lora_rank=rank, eps=0.05,
                                           lora_targets=("q", "k", "v"), loss_mode="last_pos_label_subset")
    if d != w.d_model:
        w = w.with_(d_model=d, n_heads=d // 128, n_kv_heads=d // 128, d_ffn=1024)
    room = max(k * c for k, c in ((d // 4, 3 * d), (d // 4, 2 * w.d_ffn)))       # what a pass of 256 tokens has for its partial sums
    assert M.mpz_debug_gemm_nf4_stream_units(2 * q * S, 3 * d, d, False, room) == run
    if d == 4096:
        assert M.mpz_debug_gemm_nf4_stream_units(2 * q * S, w.d_ffn, d, True, room) == 22
    frozen = M.device_random_weights(w, 1)
    masters = W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    hs = []
    for split in (True, False):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_split_k(m.handle, split)
        m.regen_noise(5, 0)
        hs.append(m.run_layers(m.embed(tokens), 0, 1, 1, S).double())
        del m
    n = 2 * q * S
    base = hs[1] - hs[1].view(2 * q, S, -1).mean(0).repeat(2 * q, 1)      # what the copies differ by
    assert hs[0].shape[0] == n and float(base.norm() / hs[1].norm()) > 0.05
    err = float((hs[0] - hs[1]).norm() / hs[1].norm())
    assert err < 8e-3, err                                 # bf16 roundings of one block that fall the other way: 4e-3 seen against 64 bits
