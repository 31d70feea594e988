"""Which kernel a GEMM over at most 256 stacked tokens takes: a host-side rule on sizes, checked without a GPU."""
import pytest

import paper_2409_15520_amd as M

ROOM = 1 << 40


# (features, K, gate and up): K = 2048 and less keeps the equal shares of K whatever the tokens; so do shapes whose equal shares
# are whole rounds of 256 blocks, and K below 4096 with more than 128 tokens
@pytest.mark.parametrize("n,k,dual,streamed", [
    (5632, 2048, True, ()), (6144, 2048, False, ()), (8192, 2048, False, ()), (2816, 1024, True, ()), (3072, 768, False, ()),
    (4096, 4096, False, ()), (4096, 11008, False, ()), (2048, 8192, False, ()), (2560, 2560, False, ()),
    (7680, 2560, False, (1, 64, 65, 128)), (6912, 2560, False, (1, 64, 65, 128)),
    (2560, 6912, False, (1, 64, 65, 128, 129, 256)), (12288, 4096, False, (1, 64, 65, 128, 129, 256)),
    (11008, 4096, True, (1, 64, 65, 128, 129, 256))])
def test_streamed_shapes(n, k, dual, streamed):
    for m in (1, 64, 65, 128, 129, 256, 257):
        assert (M.mpz_debug_gemm_stream_units(m, n, k, dual, ROOM) > 0) == (m in streamed), m


@pytest.mark.parametrize("m,n,k,dual", [(64, 12288, 4096, False), (256, 12288, 4096, False), (128, 11008, 4096, True), (96, 2560, 6912, False)])
def test_partial_sums_fit_what_they_are_given(m, n, k, dual):
    cols = 2 * n if dual else n
    for room in (0, 1, 2 * m * cols - 1, 2 * m * cols, 3 * m * cols, 9 * m * cols, ROOM):
        units = M.mpz_debug_gemm_stream_units(m, n, k, dual, room)
        if units == 0:
            assert room < 2 * m * cols                     # (two slots always do: a tile then has at most two blocks)
            continue
        nk, tiles = k // 64, (cols + 127) // 128
        owners = [{u // units for u in range(t * nk, (t + 1) * nk)} for t in range(tiles)]
        assert max(len(o) for o in owners) * m * cols <= room
        assert (tiles * nk + units - 1) // units <= 256 or room < ROOM


def test_refused_shapes_have_no_plan():
    assert M.mpz_debug_gemm_stream_units(64, 12288, 4100, False, ROOM) == 0
    assert M.mpz_debug_gemm_stream_units(0, 12288, 4096, False, ROOM) == 0
