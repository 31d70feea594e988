"""fp32 models on the 64-bit matrix instructions: parity with the oracle at the edges of the tiles (16 x 16 and 32 x 32, K by
quarters of 16), with K that no quarter divides and sequences of up to 129 tokens.  Both sides
sum in binary64 and round every stored value once, so only values next to a rounding border may differ: the bar of the
other fp32 parity tests."""
import numpy as np
import pytest

from gpu_helpers import gpu_steps, make_bundle, oracle_steps, rel_err
from small_workloads import MICRO, MINI_LLAMA, MINI_OPT

pytestmark = pytest.mark.gpu

SHAPES = {
    "d36_heads_of_6": MINI_LLAMA.with_(d_model=36, n_heads=6, n_kv_heads=3, d_ffn=52, q=1, E=1, S=15, max_seq=16, lora_rank=4),
    "d20_ffn_17_general": MINI_OPT.with_(d_model=20, n_heads=2, n_kv_heads=2, d_ffn=17, q=1, E=1, S=10, lora_rank=8),
    "S128_big_tiles": MINI_OPT.with_(d_model=64, n_heads=4, n_kv_heads=4, d_ffn=260, q=2, E=2, S=128, max_seq=129, lora_rank=12),
    "S129": MICRO.with_(q=1, E=1, S=129, max_seq=129, lora_rank=4),
    "S17_heads_of_64": MINI_LLAMA.with_(d_model=128, n_heads=2, n_kv_heads=1, d_ffn=96, q=2, E=3, S=17, max_seq=32, lora_rank=64,
                                        lora_targets=("q", "o")),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_fp32_shapes(name):
    b = make_bundle(SHAPES[name], b_std=0.02)
    Lg, Gg, Mg = gpu_steps(b, 1)
    Lo, Go, Mo = oracle_steps(b, 1)
    assert np.abs(Lg - Lo).max() <= 1e-6 * np.abs(Lo).max()
    assert rel_err(Gg[0], Go[0]) <= 1e-4
    assert rel_err(Mg, Mo) <= 1e-3
