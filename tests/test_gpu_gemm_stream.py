"""The streamed few-token GEMM (runs of K-tiles per block, partial sums per block and tile) against 64-bit products: every token
tile (64 / 128 / 256), ragged tokens and features, tiles shared by two to nine blocks, every epilogue of the reduction (the kernel
asked for by name: whether the library would choose it for a shape is test_few_token_plans's)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [1, 33, 64, 65, 128, 129, 256])
@pytest.mark.parametrize("n,k,act,f32,residual", [(4096, 4096, -1, True, True), (4100, 4096, -1, False, False), (1160, 11008, -1, True, False),
                                                  (2048, 6144, 2, False, False), (6144, 2048, 0, False, False), (50000, 2112, 1, False, False)])
def test_streamed_gemm(m, n, k, act, f32, residual):
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    nw = 2 * n if act == 2 else n
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = (torch.randn(nw, k, generator=g, device="cuda") * 0.05).bfloat16()
    b = torch.randn(nw, generator=g, device="cuda")
    r = torch.randn(m, n, generator=g, device="cuda") if residual else None
    partial = torch.empty(10 * m * nw, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    outs = []
    for _ in range(2):
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
        partial.fill_(float("nan"))                        # a slot nobody wrote would show
        M.mpz_debug_gemm_bf16_splitk(m, n, k, x.data_ptr(), w.data_ptr(), b.data_ptr(), act, None if r is None else r.data_ptr(),
                                     out.data_ptr(), f32, -1, partial.data_ptr(), partial.numel(), st)
        assert bool((out[m] == -7.0).all())
        outs.append(out[:m])
    assert torch.equal(outs[0], outs[1])                   # the slots are added in block order, whatever finished first
    y = x.double() @ w.double().t() + b.double()
    if act == 2:
        y = torch.nn.functional.silu(y[:, :n]) * y[:, n:]
    elif act == 0:
        y = torch.relu(y)
    elif act == 1:
        y = torch.nn.functional.gelu(y)
    if r is not None:
        y = y + r.double()
    err = float((outs[0].double() - y).norm() / y.norm())
    assert err < (2e-6 if f32 else 2.0 ** -8)              # fp32 sums of K products; bf16 rounding of the output


@pytest.mark.parametrize("m,n,k,act,streamed", [(64, 5632, 2048, 2, False), (33, 5632, 2048, 2, False), (200, 5632, 2048, 2, False),
                                                (128, 4096, 4096, -1, False), (256, 4096, 11008, -1, False), (128, 12288, 4096, -1, True)])
def test_chosen_kernel(m, n, k, act, streamed):
    """What the library chooses on its own has the bits of the kernel that the plan names: equal shares of K by count, or the stream."""
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    nw = 2 * n if act == 2 else n
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    w = (torch.randn(nw, k, generator=g, device="cuda") * 0.05).bfloat16()
    partial = torch.empty(16 * m * nw, device="cuda")
    assert (M.mpz_debug_gemm_stream_units(m, n, k, act == 2, partial.numel()) > 0) == streamed
    shares = M.mpz_debug_gemm_splits(m, n, k, act == 2, partial.numel())
    st = torch.cuda.current_stream().cuda_stream
    outs = []
    for ks in (0, -1, shares):
        out = torch.empty(m, n, device="cuda")
        M.mpz_debug_gemm_bf16_splitk(m, n, k, x.data_ptr(), w.data_ptr(), None, act, None, out.data_ptr(), True, ks, partial.data_ptr(),
                                     partial.numel(), st)
        outs.append(out)
    assert torch.equal(outs[0], outs[1 if streamed else 2])
    assert not torch.equal(outs[1], outs[2])               # the two cut K at different places


def test_cuts_of_k_do_not_depend_on_the_room():
    """A narrow projection of long K whose runs the partial-sum buffer limits: the same losses bit for bit from a handle made for
    just this batch, one made for more, and the library's own scratch."""
    import numpy as np
    import torch
    import paper_2409_15520_amd as M
    import workloads as W
    w = W.Workload(name="room", n_layers=3, d_model=960, n_heads=15, n_kv_heads=15, d_ffn=16384, vocab=512, max_seq=64, act="relu",
                   norm="layernorm", pos="learned", has_bias=True, tie_embeddings=True, dtype="bf16", lora_rank=8,
                   lora_targets=("q", "v"), loss_mode="next_token_all_pos", q=1, E=1, S=32, steps=1, eps=1e-2)
    assert M.mpz_debug_gemm_stream_units(64, 960, 16384, False, 4096 * 960) != M.mpz_debug_gemm_stream_units(64, 960, 16384, False, 1024 * 960)
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    tok = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    losses = []
    for E_max in (1, 16):
        m = M.ZoModel(w, frozen, masters, E_max=E_max)
        m.regen_noise(5, 0)
        losses.append(m.forward_perturbed(tok).cpu().numpy().copy())
        out = torch.zeros(2, device="cuda")
        M.mpz_forward_perturbed_noalloc(m.handle, tok.data_ptr(), None, 1, 32, out.data_ptr())
        losses.append(out.cpu().numpy().copy())
    assert np.isfinite(losses[0]).all()
    for l in losses[1:]:
        assert np.array_equal(l.view(np.uint32), losses[0].view(np.uint32)), losses
