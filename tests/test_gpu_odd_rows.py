"""Copies whose rows are no multiple of 32: an MFMA tile then holds rows of several copies.  A causal model gives a token the
same result whatever is appended after it, so such a batch is compared, bit for bit, with the same sequences padded to whole
32-row copies."""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _workload(llama, rank, q, E, S, quant="none"):
    return W.Workload(name="odd", n_layers=2, d_model=512, n_heads=8, n_kv_heads=4, d_ffn=640, vocab=600, max_seq=128,
                      act="swiglu" if llama else "relu", norm="rmsnorm" if llama else "layernorm",
                      pos="rope" if llama else "learned", has_bias=not llama, tie_embeddings=False, dtype="bf16", lora_rank=rank,
                      lora_targets=("q", "k", "v", "o") if llama else ("q", "v"), loss_mode="next_token_all_pos", q=q, E=E, S=S,
                      steps=1, eps=1e-2, weight_quant=quant)


# rows per copy 231, 21 (a tile spans three copies), 5 (eight), 99; the last tile short in all; few tokens and many
@pytest.mark.parametrize("llama,rank,q,E,S,quant", [(True, 16, 4, 3, 77, "none"), (False, 8, 4, 3, 77, "none"), (True, 8, 8, 1, 21, "none"),
                                                    (False, 16, 16, 1, 5, "none"), (True, 16, 1, 1, 99, "none"), (True, 32, 2, 3, 33, "none"),
                                                    (False, 4, 2, 3, 77, "none"), (True, 16, 2, 3, 77, "nf4")])
def test_odd_copies_equal_padded_copies(llama, rank, q, E, S, quant):
    import torch
    import paper_2409_15520_amd as M
    out = []
    padded = (S + 31) // 32 * 32
    w = _workload(llama, rank, q, E, padded, quant)
    frozen, masters = W.make_frozen_weights(w, 1), W.make_lora_masters(w, 2, b_std=0.05)
    tokens = torch.from_numpy(W.make_tokens(w, 3)).cuda()
    for length in (S, padded):
        m = M.ZoModel(w.with_(S=length), frozen, masters)
        M.mpz_debug_set_split_k(m.handle, False)           # one summation order whatever the number of rows
        m.regen_noise(5, 0)
        tok = tokens[:, :length].contiguous()
        h = m.run_layers(m.embed(tok), 0, 2, E, length).reshape(2 * q, E, length, -1)
        out.append(h[:, :, :S].clone())
        if length == S:                                    # with split K (where it applies) the same sums in another order
            M.mpz_debug_set_split_k(m.handle, True)
            again = m.run_layers(m.embed(tok), 0, 2, E, length).reshape(2 * q, E, length, -1)
            assert float((again - h).norm() / h.norm()) < 1e-2     # bf16 flips through two blocks: 4e-3 measured
    assert torch.isfinite(out[0]).all()
    assert torch.equal(out[0], out[1])
    assert not torch.equal(out[0][0], out[0][1])           # every copy has factors of its own
