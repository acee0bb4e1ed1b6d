"""The most tasks a compositor launch over 32x32 tiles may have (four per tile, sixteen for up to
fine_tile_cap tiles): an int, and within a launch's 2^32 threads, for every tile count a plan takes whose
four tasks per tile are.  Host-only."""
import pytest

from paper_2410_20686_amd import _odgs as B


@pytest.mark.parametrize("tiles", [0, 1, 255, 256, 257, 2047, 2048, 2049, 65_536, 1_000_000, 12_000_000, 12_201_612,
                                   12_300_000, 16_777_215, 16_777_216, 400_000_000, 2**29 - 1])
def test_tasks_fit_a_launch(tiles):
    cap = B.lib()._ZN4odgs13fine_tile_capEi(tiles)
    assert 0 <= cap <= tiles
    tasks = 4 * tiles + 12 * cap
    assert tasks < 2**31
    assert tasks < 2**26 or cap == 0
    if tiles <= 12_000_000:
        assert cap == min(tiles, max(256, tiles // 8))
