"""4-bit weights, 129 to 192 tokens, K in splits: the tile of all tokens (feature tiles x splits from 144 on) and the two of 128 on either side of the
rule have the bits of the dequantised weights in as many splits, with ragged tokens and features."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [128, 129, 160, 191, 192, 193])
@pytest.mark.parametrize("n,k,ks,residual", [(4100, 2560, 5, True), (4100, 2560, 4, False), (9216, 1088, 2, False), (9088, 1024, 2, False)])
def test_bits_of_the_dequantised_weights(m, n, k, ks, residual):
    import torch
    import paper_2409_15520_amd as M
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    codes = torch.randint(0, 256, (n, k // 2), dtype=torch.uint8, device="cuda", generator=g)
    absmax = (0.048 * (0.5 + torch.rand(n, k // 64, device="cuda", generator=g))).contiguous()
    w = torch.empty(n, k, dtype=torch.bfloat16, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    M.mpz_debug_dequant_nf4(codes.data_ptr(), absmax.data_ptr(), w.data_ptr(), n * k, st)
    x = torch.randn(m, k, generator=g, device="cuda").bfloat16()
    r = torch.randn(m, n, generator=g, device="cuda") if residual else None
    partial = torch.empty(ks * m * n, device="cuda")
    outs = []
    for four_bit in (True, False):
        out = torch.full((m + 1, n), -7.0, device="cuda", dtype=torch.float32 if residual else torch.bfloat16)
        partial.fill_(float("nan"))
        rp = None if r is None else r.data_ptr()
        if four_bit:
            M.mpz_debug_gemm_nf4_splitk(m, n, k, x.data_ptr(), codes.data_ptr(), absmax.data_ptr(), None, -1, rp, out.data_ptr(), residual, ks,
                                        partial.data_ptr(), partial.numel(), st)
        else:
            M.mpz_debug_gemm_bf16_splitk(m, n, k, x.data_ptr(), w.data_ptr(), None, -1, rp, out.data_ptr(), residual, ks, partial.data_ptr(),
                                         partial.numel(), st)
        assert bool((out[m] == -7.0).all())
        outs.append(out[:m])
    assert torch.equal(outs[0], outs[1])
