"""The GEMM of small outputs (32 x 32 tiles, a ring of three K-tiles of 128): bit equality with the 128 x 128 tiles, which sum in
the same order, and the 64-bit product; ragged tokens and features, one to seven K-tiles, every epilogue, operands that
do not begin on 16 bytes (which keep the other tiles)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(1, 4, 128), (31, 36, 256), (33, 28, 384), (97, 768, 768), (64, 100, 896), (384, 520, 128)])
@pytest.mark.parametrize("act,f32,shift", [(-1, True, 0), (0, False, 0), (1, True, 0), (-1, False, 4)])
def test_small_tiles(m, n, k, act, f32, shift):
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn(m * k + shift, generator=g, device="cuda").bfloat16()[shift:].view(m, k)
    w = (torch.randn(n, k, generator=g, device="cuda") * 0.05).bfloat16()
    b = torch.randn(n, generator=g, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    outs = []
    for cfg in (14, 1):
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if f32 else torch.bfloat16)
        M.mpz_debug_gemm_bf16(m, n, k, x.data_ptr(), w.data_ptr(), b.data_ptr(), act, out.data_ptr(), f32, st, cfg)
        assert bool((out[m] == -7.0).all())
        outs.append(out[:m])
    assert torch.equal(outs[0], outs[1])
    y = x.double() @ w.double().t() + b.double()
    y = torch.relu(y) if act == 0 else torch.nn.functional.gelu(y) if act == 1 else y
    assert float((outs[0].double() - y).norm() / y.norm()) < (2e-6 if f32 else 2.0 ** -8)   # fp32 sums; bf16 output
