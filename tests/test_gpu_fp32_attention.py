"""fp32 models: attention on the 64-bit matrix instructions at the edges of its tiles of 16 queries and keys, against the oracle on
the same operands, and tokens that are not numbers behind a query; linears on tiles of 48, ragged in rows, columns and K."""
import numpy as np
import pytest

from gpu_helpers import gpu_model, gpu_steps, make_bundle, oracle_steps, rel_err
from oracle.model import _attention
from oracle.precision import Precision
from small_workloads import MINI_LLAMA, MINI_OPT

pytestmark = pytest.mark.gpu
F32 = Precision("f32")


def _attend(H, Hkv, dh, S, qkv, n_seq):
    import torch
    import paper_2409_15520_amd as M
    w = MINI_LLAMA.with_(d_model=H * dh, n_heads=H, n_kv_heads=Hkv, d_ffn=64, q=1, E=1, S=S, max_seq=max(S, 2), n_layers=1)
    m = gpu_model(make_bundle(w))
    x = torch.from_numpy(qkv).cuda()
    out = torch.full((n_seq * S + 1, H * dh), -7.0, device="cuda")
    M.mpz_debug_attention(m.handle, x.data_ptr(), n_seq, S, out.data_ptr())
    out = out.cpu().numpy()
    assert (out[n_seq * S] == -7.0).all()
    return out[:n_seq * S]


def _operands(H, Hkv, dh, S, n_seq):
    rng = np.random.default_rng(S * dh)
    return [(2.0 * rng.standard_normal((n_seq, S, h, dh))).astype(np.float32) for h in (H, Hkv, Hkv)]


# (heads of 48 and 129 tokens: the shape-agnostic kernel)
@pytest.mark.parametrize("H,Hkv,dh", [(4, 4, 32), (6, 2, 64), (2, 1, 48)])
@pytest.mark.parametrize("S", [2, 15, 16, 17, 32, 33, 64, 65, 96, 127, 128, 129])
def test_attention(H, Hkv, dh, S):
    q, k, v = _operands(H, Hkv, dh, S, 3)
    qkv = np.concatenate([t.reshape(3 * S, -1) for t in (q, k, v)], axis=1)
    got = _attend(H, Hkv, dh, S, qkv, 3)
    want = _attention(q.astype(np.float64), k.astype(np.float64), v.astype(np.float64), H, Hkv, F32).reshape(3 * S, -1).astype(np.float32)
    # 64-bit sums on both sides: a probability or result next to a rounding border may fall the other way (one unit of fp32)
    assert np.abs(got - want).max() <= 2.0 ** -22 * np.abs(v).max()
    assert (got != want).mean() < 1e-3


# the first lengths that are taken, and the last that is not
@pytest.mark.parametrize("S", [7, 8, 9])
def test_short_sequences(S):
    test_attention(6, 2, 64, S)


@pytest.mark.parametrize("S,bad", [(16, 9), (33, 32), (70, 50)])
def test_tokens_behind_a_query_do_not_reach_it(S, bad):
    H, dh = 2, 32
    q, k, v = _operands(H, H, dh, S, 1)
    clean = _attend(H, H, dh, S, np.concatenate([t.reshape(S, -1) for t in (q, k, v)], axis=1), 1)
    for t in (q, k, v):
        t[:, bad] = np.inf
    k[:, bad, 1] = np.nan
    got = _attend(H, H, dh, S, np.concatenate([t.reshape(S, -1) for t in (q, k, v)], axis=1), 1)
    assert np.array_equal(got[:bad], clean[:bad]) and not np.isfinite(got[bad]).any()


def test_linears_on_tiles_of_48():
    """760 rows in copies of 190 (a tile of 16 spans two), 756 and 760 columns, K = 252."""
    w = MINI_OPT.with_(d_model=252, n_heads=6, n_kv_heads=6, d_ffn=760, q=2, E=2, S=95, max_seq=96, lora_rank=8, n_layers=1)
    b = make_bundle(w, b_std=0.02)
    Lg, Gg, Mg = gpu_steps(b, 1)
    Lo, Go, Mo = oracle_steps(b, 1)
    assert np.abs(Lg - Lo).max() <= 1e-6 * np.abs(Lo).max()
    assert rel_err(Gg[0], Go[0]) <= 1e-4
    assert rel_err(Mg, Mo) <= 1e-3
