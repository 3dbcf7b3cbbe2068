"""The tile shapes the many-row product plans are the ones its GPU test runs."""
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
