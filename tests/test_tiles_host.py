"""The tile shapes the many-row product plans are the ones its GPU test runs."""
import pytest

from tests import _tiles as T


def test_planned_tiles_are_tested_tiles():
    tiles = set(T.TILES)
    seen = set()
    for R in (25, 32, 33, 41, 64, 65, 96, 128, 129, 164, 192, 193, 222, 256, 257, 320, 511, 700, 1024, 1301, 2047, 2048):
        for N in (16, 48, 512, 1040, 2048, 2560, 4096, 5120, 6144, 10240, 12288, 15360, 16400, 22016, 27648, 32000):
            for K in (32, 96, 1024, 2048, 4096, 5120, 11008, 13824):
                for part in (0, 256 ** 3):
                    t = T.planned(R, N, K, T.RESID, part)
                    assert t[:3] in tiles, (R, N, K, t)
                    assert 1 <= t[3] <= 8 and (part or t[3] == 1)
                    seen.add(t[:3])
    assert seen == tiles, f"never planned: {sorted(tiles - seen)}"


def test_passes_of_up_to_32_rows_take_tiles_of_32():
    for N, K in ((27648, 5120), (32000, 4096), (57344, 8192), (5120, 13824)):
        assert all(T.planned(R, N, K)[1] == 0 for R in (25, 29, 32)) and T.planned(33, N, K)[1] == 1


# measured on both kernels at 256 compute units; terms = the shortest reduction for which the many-row kernel is the faster one
@pytest.mark.parametrize("R,N,terms", [(64, 1024, 3072), (57, 2048, 3072), (56, 1024, 4096), (40, 1024, 4096), (32, 1024, 5120), (64, 4096, 4096), (40, 4096, 5120),
                                       (32, 4096, 8192), (25, 6144, 5120), (64, 6144, 3072), (32, 8192, 10240), (33, 8192, 5120), (40, 10240, 5632), (25, 10240, 8192),
                                       (33, 12288, 10240), (48, 12288, 8192), (64, 12288, 5120), (25, 15360, 5120)])
def test_route_of_25_to_64_rows(R, N, terms):
    assert T.many_rows(R, N, terms) and not T.many_rows(R, N, terms - 32)
    assert not T.many_rows(R, N, 32 * 1024, part_floats=0)     # nothing to cut with


def test_route_of_other_rows():
    for N, K in ((16, 32), (1024, 256), (12288, 4096), (32000, 13824)):
        assert T.many_rows(65, N, K, 0) and T.many_rows(256, N, K) and not T.many_rows(24, N, K)
    assert not T.many_rows(25, 12288, 13824) and T.many_rows(25, 16384, 32, 0)
