"""Which tile a GEMM takes: the library's rules on sizes, asked without a GPU.  Tiles by number: 6 = 256 x 256, 11 = 192 x 128, 12 and 1 =
128 x 128, 15 = the same for rotated heads of 128, 9 = 128 x 64, 10 = 64 x 64, 14 = 32 x 32; -1 = refused."""
import pytest

import paper_2409_15520_amd as M
from dispatch_program import ask


# one key-value head (two of 64): 128 rotated columns over.  K of 4096 keeps the wide tile, whose launch refuses the rotation
@pytest.mark.parametrize("bits", [16, 8])
@pytest.mark.parametrize("m,n,k,rope,dh,tile", [(10240, 2304, 2048, 2176, 128, 15), (10240, 2304, 2048, 2176, 64, 12), (5120, 2304, 2048, 2176, 64, 12),
                                                (24576, 2304, 2048, 2176, 64, 12), (10240, 2304, 2048, 2048, 64, 6), (10240, 2560, 2048, 2304, 64, 6),
                                                (10240, 4352, 4096, 4224, 128, -1), (10240, 4608, 4096, 4352, 128, 6)])
def test_rotated_columns_that_end_inside_a_wide_tile(m, n, k, rope, dh, tile, bits):
    assert ask([f"tile {m} {n} {k} {bits} {rope} {dh}"]) == [tile]


# 256 x 256 tiles, 128 x 128 ones of the same product: 144, 480 and 504 (rows that fill part of a wide tile); 130, 516; 144, 576; 256, 1024;
# two rounds: 264, 1056; 305, 1210; 320, 1280; K of 1024 has no second round, K of 768 no first
@pytest.mark.parametrize("m,n,k,wide", [(576, 12288, 4096, False), (640, 12288, 4096, False), (896, 9216, 3072, False), (2560, 3328, 4096, True),
                                        (3072, 3072, 1024, True), (4096, 4096, 1024, True), (3072, 3072, 768, False),
                                        (2816, 6144, 2048, False), (15616, 1280, 2048, False), (4096, 5120, 2048, True), (4096, 5120, 1024, False),
                                        (8192, 4096, 768, True)])
def test_wide_tiles_by_the_half_rounds_of_small_ones(m, n, k, wide):
    assert (ask([f"tile {m} {n} {k} 16 0 0"])[0] == 6) == wide


# gate and up: wide tiles, 128 x 128 ones: 132, 220; 132, 264; 258, 430; 258, 516; 160, 240; 128, 256; 128, 224; 256, 512
@pytest.mark.parametrize("m,n,k,wide", [(576, 5632, 2048, False), (768, 5632, 2048, True), (640, 11008, 4096, False), (768, 11008, 4096, True),
                                        (384, 10240, 4096, False), (1024, 4096, 2048, False), (896, 4096, 1536, False), (1024, 8192, 1024, True),
                                        (768, 11008, 1024, False), (768, 5632, 768, False), (4096, 11008, 768, True)])
def test_gate_and_up_wide_where_small_tiles_need_more_rounds(m, n, k, wide):
    assert (ask([f"tile {m} {n} {k} 16 -1 0"])[0] == 6) == wide


# int8: one round of wide tiles against two, three (513 to 768 small tiles) and four of small ones, two against five and six
@pytest.mark.parametrize("m,n,k,wide", [(2048, 4096, 4096, False), (576, 12288, 4096, False), (1024, 12288, 4096, True), (2304, 4096, 2048, True),
                                        (3072, 3072, 1536, False), (4096, 5120, 4096, False), (8192, 2560, 2048, False), (5632, 4096, 4096, True),
                                        (3072, 7680, 2560, True), (8192, 4096, 1024, True)])
def test_int8_wide_tiles_by_rounds(m, n, k, wide):
    assert (ask([f"tile {m} {n} {k} 8 0 0"])[0] == 6) == wide


@pytest.mark.parametrize("m,n,k,wide", [(384, 10240, 4096, False), (512, 11008, 4096, True), (640, 11008, 4096, False), (768, 11008, 4096, True),
                                        (896, 4096, 2048, False), (768, 5632, 2048, True), (768, 5632, 1536, False)])
def test_int8_gate_and_up_wide_where_small_tiles_need_more_rounds(m, n, k, wide):
    assert (ask([f"tile {m} {n} {k} 8 -1 0"])[0] == 6) == wide


# 144 whole tiles of 240 and 252 halves, of 288; 192; 132 of 264
@pytest.mark.parametrize("m,n,k,tile", [(288, 6144, 2048, 9), (300, 6144, 8192, 9), (448, 4608, 1536, 9), (384, 6144, 2048, 12), (512, 6144, 2048, 12),
                                        (3072, 768, 3072, 12), (1408, 1536, 2048, 9)])
def test_halves_of_tiles_that_fit_the_cus(m, n, k, tile):
    assert ask([f"tile {m} {n} {k} 16 0 0"]) == [tile]


@pytest.mark.parametrize("m,n,k,tile", [(320, 2048, 512, 14), (384, 2048, 512, 14), (320, 2048, 768, 10), (320, 2048, 2048, 10), (320, 2048, 4096, 14),
                                        (288, 2048, 4096, 10), (384, 2048, 5632, 14), (320, 2048, 8192, 10), (256, 2048, 2048, 14), (416, 2048, 4096, 10)])
def test_the_smallest_tiles_of_wide_outputs(m, n, k, tile):
    assert ask([f"tile {m} {n} {k} 16 0 0"]) == [tile]


# weights that the last-level cache holds and that it does not (256 MiB, 250, 449; gate and up 224 and 432): the 256 x 256 tile (-1) stays unless the
# fitted ones (20 + shape) gain much; not where the 128 x 128 ones were the other choice
@pytest.mark.parametrize("m,n,k,dual,tile", [(576, 16384, 4096, False, 21), (576, 16384, 8192, False, -1), (768, 16384, 8192, False, -1), (1152, 16384, 8192, False, 23),
                                             (384, 16384, 8192, False, 23), (288, 32000, 4096, False, -1), (1152, 32000, 4096, False, -1), (320, 28672, 8192, False, -1),
                                             (1152, 28672, 8192, False, 24), (576, 14336, 4096, True, 23), (640, 16384, 6912, True, -1)])
def test_fitted_tiles_and_weights_past_the_last_level_cache(m, n, k, dual, tile):
    assert M.mpz_debug_gemm_fitted_tile(m, n, k, dual) == tile
