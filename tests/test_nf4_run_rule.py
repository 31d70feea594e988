"""Which 4-bit projections over at most 256 stacked tokens the streamed kernel takes, and in which runs (no GPU)."""
import pytest

from dispatch_program import ask


def runs(m, n, k, rows=1 << 20):
    return ask([f"nf4_run {m} {n} {k} {rows}"])[0]


# whole runs: from 18 K-tiles on up to 128 tokens, 12 up to 192, 14 up to 256; runs that cross tiles: also where shares of K leave CUs
# idle (17408, 22016 and 10240 columns) and not where they are full (16384 x 4288, 21504 x 3904, 12288 x 4288) unless the runs are long
@pytest.mark.parametrize("n,k,run,tokens", [
    (12288, 4096, 16, (129, 192, 193, 256)), (22016, 4096, 22, (1, 64, 128, 129, 192, 193, 256)), (4096, 4096, 0, ()), (4096, 11008, 0, ()),
    (8192, 6144, 12, (129, 192)), (4096, 14336, 14, (129, 192, 193, 256)), (8192, 8192, 16, (129, 192, 193, 256)),
    (5120, 13824, 18, (1, 64, 128, 129, 192, 193, 256)), (17408, 4288, 18, (1, 64, 128, 129, 192, 193, 256)),
    (10240, 8192, 20, (1, 64, 128, 129, 192, 193, 256)), (16384, 4288, 17, (129, 192)), (21504, 3904, 21, (129, 192, 193, 256)),
    (12288, 4288, 13, (129, 192)), (17280, 3200, 14, (129, 192, 193, 256)), (16384, 2048, 0, ()), (57344, 8192, 128, (1, 64, 128, 129, 192, 193, 256))])
def test_runs(n, k, run, tokens):
    for m in (1, 64, 128, 129, 192, 193, 256):
        assert runs(m, n, k) == (run if m in tokens else 0), m
    assert runs(257, n, k) == 0


@pytest.mark.parametrize("m,n,k", [(192, 12288, 4096), (256, 22016, 4096), (64, 22016, 4096), (192, 2048, 16384)])
def test_partial_sums_fit_what_they_are_given(m, n, k):
    nk, tiles = k // 64, (n + 255) // 256
    for rows in (0, m, 2 * m - 1, 2 * m, 3 * m, 4 * m, 5 * m, 16 * m):
        u = runs(m, n, k, rows)
        if u:
            owners = [{i // u for i in range(t * nk, (t + 1) * nk)} for t in range(tiles)]
            assert max(len(o) for o in owners) * m <= rows
            assert (tiles * nk + u - 1) // u >= 192        # little room never leaves a quarter of the CUs idle
