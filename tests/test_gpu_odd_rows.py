"""Copies whose rows are no multiple of 32, and the other adapted linears that the bf16 matrix kernels do not take: every sum is
the binary32 chain of the shape-agnostic kernels, term by term, so the results are theirs bit for bit.  (Two-point
differences of small batches amplify another order of summation beyond the bound of a step's masters.)"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _workload(llama, d, heads, kv, rank, q, E, S, targets, quant="none"):
    return W.Workload(name="odd", n_layers=1, d_model=d, n_heads=heads, n_kv_heads=kv, d_ffn=640, vocab=600, max_seq=256,
                      act="swiglu" if llama else "relu", norm="rmsnorm" if llama else "layernorm",
                      pos="rope" if llama else "learned", has_bias=not llama, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                      lora_targets=tuple(targets), loss_mode="next_token_all_pos", q=q, E=E, S=S, steps=1, eps=1e-2, weight_quant=quant)


# rows per copy 231, 21 (a tile of 32 spans three copies), 2 (sixteen), 99, 33, 32; the last tile short; K of one and of many
# K-tiles of 64; output widths and segments that begin and end inside a tile; few rows and many; few columns of a bottleneck and
# more than the matrix kernels take (rank 64); K = 192 and 320 also for whole copies
@pytest.mark.parametrize("d,heads,kv,rank,q,E,S,targets", [
    (512, 8, 4, 16, 4, 3, 77, "qkv"), (512, 8, 4, 8, 8, 1, 21, "qv"), (64, 4, 2, 4, 16, 1, 2, "kv"), (2048, 16, 2, 16, 1, 1, 99, "qv"),
    (512, 8, 8, 32, 2, 3, 33, "qkv"), (192, 8, 1, 12, 3, 1, 33, "qkv"), (320, 10, 10, 64, 2, 1, 32, "qkv"), (768, 12, 12, 8, 1, 5, 45, "q")])
def test_projection_has_the_bits_of_the_shape_agnostic_kernels(d, heads, kv, rank, q, E, S, targets):
    import torch
    import paper_2409_15520_amd as M
    w = _workload(False, d, heads, kv, rank, q, E, S, targets)
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    T, n = 2 * q * E * S, d + 2 * w.d_kv
    x = torch.randn(T, d, generator=torch.Generator(device="cuda").manual_seed(d + T), device="cuda").bfloat16()
    outs = []
    for simple in (False, True):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_kernel_path(m.handle, simple)
        m.regen_noise(5, 0)
        out = torch.full((T + 1, n), -7.0, device="cuda")
        M.mpz_debug_qkv_projection(m.handle, x.data_ptr(), 0, E, S, out.data_ptr())
        assert bool((out[T] == -7.0).all())
        outs.append(out[:T])
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1])
    y = outs[0].reshape(2 * q, E * S, n)
    assert not torch.equal(y[0], y[1])                     # every copy has factors of its own


# enough rows and columns for the larger wave tile, which ends inside rows, columns and segments (1120 columns, segments from 1088 and
# 1104); many blocks of the bottleneck, whole pairs of its K-tiles and not
@pytest.mark.parametrize("d,heads,q,E,S,rank", [(1088, 68, 4, 3, 81, 16), (1088, 68, 16, 1, 77, 20), (512, 8, 16, 7, 33, 24)])
def test_many_rows_have_the_bits_of_the_shape_agnostic_kernels(d, heads, q, E, S, rank):
    test_projection_has_the_bits_of_the_shape_agnostic_kernels(d, heads, 1, rank, q, E, S, "qkv")


# widths of 32 modulo 64: a bottleneck whose last K-tile is half outside (one K-tile and many), its last rows those of the operand
@pytest.mark.parametrize("d,heads,kv,rank,q,E,S,targets", [(32, 2, 1, 4, 2, 1, 33, "qkv"), (96, 4, 4, 8, 4, 3, 77, "qv"), (96, 4, 2, 20, 2, 1, 33, "qkv"),
                                                           (288, 4, 4, 16, 2, 1, 5, "qv"), (352, 8, 2, 8, 2, 3, 45, "qkv"), (1312, 8, 8, 16, 2, 1, 99, "q")])
def test_widths_of_half_a_k_tile_have_the_bits_of_the_shape_agnostic_kernels(d, heads, kv, rank, q, E, S, targets):
    test_projection_has_the_bits_of_the_shape_agnostic_kernels(d, heads, kv, rank, q, E, S, targets)


# columns of several targets in one tile of 16: all in one, a target that ends inside one, one that spans two, a last tile with 4 and 12
# columns; outputs of the same columns as one target at a time
@pytest.mark.parametrize("rank,targets", [(4, "qv"), (4, "qkv"), (8, "qkv"), (12, "qk"), (12, "qkv"), (20, "kv"), (28, "qkv")])
def test_targets_in_one_tile_have_the_bits_of_the_shape_agnostic_kernels(rank, targets):
    test_projection_has_the_bits_of_the_shape_agnostic_kernels(288, 4, 2, rank, 2, 3, 45, targets)


# a block whose every other part takes the same kernels either way (d = 320, heads of 32) and whose feed-forward adds exact
# zeros: norm, q/k/v with rotary staging or not, attention, output projection with residual; 4-bit weights once per pass
@pytest.mark.parametrize("llama,rank,q,E,S,quant", [(True, 16, 4, 3, 77, "none"), (False, 8, 4, 3, 77, "none"), (True, 32, 2, 3, 33, "none"),
                                                    (False, 4, 16, 1, 5, "none"), (True, 16, 2, 3, 77, "nf4"), (False, 16, 2, 1, 21, "nf4")])
def test_block_has_the_bits_of_the_shape_agnostic_kernels(llama, rank, q, E, S, quant):
    import torch
    import paper_2409_15520_amd as M
    w = _workload(llama, 320, 10, 5, rank, q, E, S, "qkvo", quant)
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    lw = frozen["layers"][0]
    lw["s_down" if quant == "nf4" else "w_down"] = np.zeros_like(lw["s_down" if quant == "nf4" else "w_down"])
    if lw["b_down"] is not None:
        lw["b_down"] = np.zeros_like(lw["b_down"])
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    outs = []
    for simple in (False, True):
        m = M.ZoModel(w, frozen, masters)
        M.mpz_debug_set_kernel_path(m.handle, simple)
        m.regen_noise(5, 0)
        outs.append(m.run_layers(m.embed(tokens), 0, 1, E, S).reshape(2 * q, E * S, -1).clone())
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1])
    assert not torch.equal(outs[0][0], outs[0][1])


def test_int8_weights_refuse_odd_copies():
    """No kernel that keeps this order reads int8 codes; a pass over single blocks refuses such copies as the whole pass does."""
    import torch
    import paper_2409_15520_amd as M
    w = _workload(True, 512, 8, 4, 16, 2, 1, 33, "qv", "int8")
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05))
    m.regen_noise(5, 0)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    h = m.embed(tokens)
    with pytest.raises(M.MpzError) as e:
        m.run_layers(h, 0, 1, 1, 33)
    assert e.value.status == 3                             # MPZ_ERR_SHAPE


# few tokens: the linears without adapters split K (or, 4-bit, look their codes up) whatever the rows of a copy; the adapted ones
# don't.  Another order of the same fp32 sums: bf16 flips through one block, 4e-3 at most as measured for whole copies
@pytest.mark.parametrize("q,E,S,quant", [(1, 1, 33, "none"), (2, 1, 21, "none"), (8, 1, 5, "nf4"), (1, 3, 33, "nf4")])
def test_few_tokens_of_odd_copies(q, E, S, quant):
    import torch
    import paper_2409_15520_amd as M
    w = _workload(True, 2048, 16, 4, 16, q, E, S, "qkvo", quant).with_(d_ffn=5632)
    T = 2 * q * E * S
    assert T % 32 and M.mpz_debug_gemm_splits(T, 5632, 2048, True, 1 << 40) >= 2 and M.mpz_debug_gemm_splits(T, 2048, 5632, False, 1 << 40) >= 2
    m = M.ZoModel(w, W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05))
    m.regen_noise(5, 0)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    outs = []
    for split in (True, False):
        M.mpz_debug_set_split_k(m.handle, split)
        outs.append(m.run_layers(m.embed(tokens), 0, 1, E, S).clone())
    assert torch.isfinite(outs[0]).all()
    err = float((outs[0] - outs[1]).norm() / outs[1].norm())
    print(f"\nodd few tokens q {q} E {E} S {S} {quant}: {err:.2e}")
    assert 0 < err < 8e-3
