"""Rules of the attention kernel (no GPU).  Where the attention of one key chunk keeps its scores and where it computes them twice (no GPU): 128 keys with heads of 64, 64
with heads of 128, and there operands and results of some 300 MB unless the heads share keys.  From which length on a sequence's rows are more than the offsets into one buffer reach."""
import pytest

from dispatch_program import ask


@pytest.mark.parametrize("n,S,H,kv,dh,keeps", [(8, 128, 32, 4, 64, True), (8, 129, 32, 4, 64, False), (128, 128, 32, 4, 64, True), (256, 112, 32, 4, 64, True),
                                               (256, 128, 32, 4, 64, True), (512, 96, 16, 8, 64, True), (8, 64, 20, 20, 128, True), (8, 65, 20, 20, 128, False),
                                               (128, 64, 20, 20, 128, True), (256, 64, 20, 20, 128, False), (512, 64, 16, 2, 128, True)])
def test_sizes(n, S, H, kv, dh, keeps):
    assert ask([f"attention_keeps {n} {S} {H} {kv} {dh}"]) == [keeps]


# blocks of 256 queries (sequences x heads x blocks of one): few, the last 256 of them half there and a little more, many; lengths around
# three quarters of a block
@pytest.mark.parametrize("n,S,H,dh,eight", [(2, 256, 32, 64, False), (4, 256, 32, 64, False), (5, 256, 32, 64, True), (8, 256, 32, 64, True), (9, 256, 32, 64, False),
                                            (12, 256, 32, 64, False), (13, 256, 32, 64, True), (16, 256, 32, 64, True), (20, 200, 32, 64, False), (21, 200, 32, 64, True),
                                            (2, 512, 32, 64, False), (3, 512, 32, 64, True), (6, 512, 32, 64, False), (12, 512, 32, 64, True), (128, 512, 32, 64, True),
                                            (40, 191, 4, 64, False), (40, 192, 4, 64, True), (40, 257, 4, 64, False), (20, 447, 4, 64, False), (20, 448, 4, 64, True),
                                            (8, 128, 32, 64, False), (8, 256, 32, 128, False)])
def test_eight_waves(n, S, H, dh, eight):
    assert ask([f"attention_eight {n} {S} {H} {dh}"]) == [eight]


@pytest.mark.parametrize("H,kv,dh", [(32, 32, 128), (32, 4, 64), (128, 128, 64), (128, 8, 128)])
def test_sequences_that_one_buffer_does_not_reach(H, kv, dh):
    row = (H + 2 * kv) * dh * 2
    lo, hi = 2, 1 << 24                                    # the longest near sequence, the first far one
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if ask([f"attention_far {mid} {H} {kv} {dh}"])[0] else (mid, hi)
    piece = 64 if dh == 64 else 32
    past = -(-lo // piece) * piece - 1                     # the last row that a piece begins to ask for
    assert (lo - 1) * row + kv * dh * 2 + dh * 2 <= 0x7ff00000, "the size of the buffer, below the offsets that mean past the end"
    assert past * row + kv * dh * 2 + dh * 2 < 1 << 31, "offsets of the last piece"
    assert (lo + 70) * row > 0x7ff00000                    # and no sooner than that asks for
    assert ask([f"attention_far {s} {H} {kv} {dh}" for s in (2, 512, lo - 1, lo, hi, hi + 1, 174764 * 24576 // row, 1 << 24)]) == [0] * 4 + [1] * 4
