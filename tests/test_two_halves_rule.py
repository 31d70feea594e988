"""Which sizes run as two halves on two streams (no GPU): weight_quant 0 = bf16, 1 = int8.  Every size of 3072 tokens or more below d = 2048, and
every int8 one but 3840 tokens, was timed both ways, and the answer is the faster one (one pass over two halves, 4 layers, in the comments)."""
import pytest

from dispatch_program import ask

OPT = {768: "768 2304 3072 0", 1536: "1536 4608 6144 0", 2048: "2048 6144 8192 0", 2560: "2560 7680 6912 0", 3072: "3072 9216 12288 0"}
LLAMA = {1024: "1024 2048 2816 1", 2048: "2048 2560 5632 1", 3072: "3072 5120 8192 1"}


@pytest.mark.parametrize("shape,quant,tokens,halves", [
    (LLAMA[1024], 0, 3008, False), (LLAMA[1024], 0, 3072, False),         # too few tokens; 0.96
    (LLAMA[1024], 0, 4096, False), (LLAMA[1024], 0, 4608, True), (LLAMA[1024], 0, 6144, False), (LLAMA[1024], 0, 6656, True),   # 0.91, 1.07, 0.92, 1.07
    (LLAMA[1024], 0, 8192, False), (LLAMA[1024], 0, 9216, True), (LLAMA[1024], 0, 14848, False),                                # 0.98, 1.14, 0.99
    (OPT[768], 0, 7168, False), (OPT[768], 0, 8192, False), (OPT[768], 0, 8704, True), (OPT[768], 0, 10752, False),             # 0.93, 0.96, 1.05, 0.97
    (OPT[768], 0, 11264, True), (OPT[768], 0, 16384, False), (OPT[1536], 0, 3584, False), (OPT[1536], 0, 5632, True),           # 1.11, 0.96, 0.95, 1.13
    (LLAMA[1024], 1, 5120, False), (LLAMA[1024], 1, 4096, False), (LLAMA[1024], 1, 9216, True), (OPT[768], 1, 7168, False),     # 0.99, 0.88, 1.14, 0.91
    (OPT[768], 1, 8192, True), (OPT[1536], 1, 3584, False), (OPT[1536], 1, 4096, True),                                         # 1.06, 0.88, 1.08
    # both wide projections a little over one round of 256-wide tiles; the tokens and widths next to them, and gate and up
    (OPT[2560], 0, 2304, False), (OPT[2560], 0, 2560, True), (OPT[2560], 0, 2816, False), (OPT[2048], 0, 3072, False), (OPT[3072], 0, 2048, False),
    (LLAMA[2048], 0, 3072, False), (LLAMA[3072], 0, 3328, False),
    (OPT[2560], 1, 2048, False), (OPT[2560], 1, 2560, True), (OPT[2560], 1, 3328, True), (OPT[2560], 1, 3840, False),           # 0.86, 1.06, 1.06
    (OPT[2048], 1, 2560, False), (OPT[2048], 1, 2816, False), (OPT[2048], 1, 3328, True), (OPT[2048], 1, 3584, False),          # 0.96, 0.94, 1.05, 1.01
    (OPT[3072], 1, 1536, False), (OPT[3072], 1, 2048, True), (OPT[3072], 1, 2560, False),                                       # 0.96, 1.08, 1.00
    (LLAMA[2048], 1, 4608, False), (LLAMA[3072], 1, 2048, False),
    # never so few tokens that a half would split K (widths that have many tiles all the same)
    ("2048 6144 66048 0", 1, 512, False), ("2048 6144 33024 0", 1, 512, False)])
def test_sizes(shape, quant, tokens, halves):
    assert ask([f"two_halves {shape} {quant} {tokens}"]) == [halves]
