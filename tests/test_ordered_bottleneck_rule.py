"""Which bottlenecks of odd copies the fp32 matrix instructions take, and in how many blocks (no GPU)."""
import pytest

from dispatch_program import ask


@pytest.mark.parametrize("k,taken", [(32, True), (64, True), (96, True), (288, True), (352, True), (1312, True), (2048, True), (48, False), (100, False)])
def test_widths(k, taken):
    """Whole pieces of 32 columns, 32 modulo 64 among them."""
    assert (ask([f"lora_down_ordered {k} 8 2 33 4"])[0] > 0) == taken
