"""Pre-norm and bottleneck in one kernel at d_model 2048 (eight waves: two halves of the bottleneck's columns, four rows a wave)
against the two kernels it stands for: the same arithmetic in the same order, so the same bits."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_model, make_bundle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,rank,targets,S", [
    ("c4_llama1p1b", 16, ("q", "k", "v"), 160),           # 48 columns: the second half of them part-empty; RMS norm
    ("c4_llama1p1b", 16, ("q", "k", "v", "o"), 32),       # two blocks of rows
    ("c3_opt1p3b", 16, ("q", "k", "v"), 288),             # layer norm with its bias
])
def test_wide_fused_norm_and_bottleneck_changes_no_bit(base, rank, targets, S):
    import torch
    import paper_2409_15520_amd as M
    w = W.get_workload(base).with_(n_layers=2, q=1, E=1, S=S, vocab=4096, max_seq=288, lora_rank=rank, lora_targets=targets)
    b = make_bundle(w, b_std=0.05)
    m = gpu_model(b)
    tok = torch.from_numpy(b["tokens"]).cuda()
    lab = torch.from_numpy(b["labels"]).cuda()
    out = []
    for enable in (True, False):
        M.mpz_debug_set_fused_norm_lora(m.handle, enable)
        m.regen_noise(3456, 0)
        out.append(m.forward_perturbed(tok, lab).cpu().numpy().copy())
    assert np.array_equal(out[0].view(np.uint32), out[1].view(np.uint32)), out
