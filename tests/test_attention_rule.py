"""Where the attention of one key chunk keeps its scores and where it computes them twice (no GPU): chunks of 128 keys with heads of 64, of 64
with heads of 128, and operands and results of some 300 MB."""
import pytest

from dispatch_program import ask


@pytest.mark.parametrize("n,S,H,kv,dh,keeps", [(8, 128, 32, 4, 64, True), (8, 129, 32, 4, 64, False), (128, 128, 32, 4, 64, True), (256, 112, 32, 4, 64, True),
                                               (256, 128, 32, 4, 64, False), (512, 96, 16, 8, 64, False), (8, 64, 20, 20, 128, True), (8, 65, 20, 20, 128, False),
                                               (128, 64, 20, 20, 128, True), (256, 64, 20, 20, 128, False), (512, 64, 16, 2, 128, True)])
def test_sizes(n, S, H, kv, dh, keeps):
    assert ask([f"attention_keeps {n} {S} {H} {kv} {dh}"]) == [keeps]
