"""Which bottlenecks of odd copies the fp32 matrix instructions take, and in how many blocks (no GPU)."""
import pytest

from dispatch_program import ask


@pytest.mark.parametrize("k,taken", [(32, True), (64, True), (96, True), (288, True), (352, True), (1312, True), (2048, True), (48, False), (100, False)])
def test_widths(k, taken):
    """Whole pieces of 32 columns, 32 modulo 64 among them."""
    assert (ask([f"lora_down_ordered {k} 8 2 33 4"])[0] > 0) == taken


@pytest.mark.parametrize("rank,targets", [(4, 1), (4, 2), (4, 3), (8, 2), (8, 3), (12, 3), (16, 1), (16, 3), (20, 2), (24, 3), (64, 3)])
def test_targets_share_tiles_of_columns(rank, targets):
    """16 columns a block, of all targets side by side: 4 copies of 77 rows are two tiles of rows each."""
    assert ask([f"lora_down_ordered 768 {rank} {targets} 77 4"])[0] == 4 * 2 * ((rank * targets + 15) // 16)


def test_a_refused_lds_limit_is_not_a_launch():
    """Without a device the kernel's LDS limit cannot be raised: nothing is launched (the caller takes the shape-agnostic kernel)."""
    assert ask(["lora_down_ordered_launch 768 8 2 77 4", "lora_down_ordered_launch 96 8 2 77 4"]) == [0, 0]
