"""Which attention of fp32 models the 64-bit matrix instructions take (no GPU): by the tokens of a sequence, whatever their number."""
import pytest

from dispatch_program import ask


@pytest.mark.parametrize("S,dh,taken", [(1, 64, False), (4, 64, False), (7, 32, False), (8, 32, True), (8, 64, True), (128, 64, True), (129, 64, False),
                                        (64, 48, False), (64, 128, False)])
def test_tokens(S, dh, taken):
    assert ask([f"attention_f64 {n} {S} 12 {dh}" for n in (1, 4, 256)]) == [taken] * 3


def test_as_many_blocks_as_a_launch_has_threads():
    assert ask(["attention_f64 174762 128 12 64", "attention_f64 174763 128 12 64"]) == [1, 0]
