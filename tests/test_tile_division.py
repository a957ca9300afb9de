"""CPU: the multipliers by which the kernels divide tile ids by the map side and the
palette size are exact for every id, with the hardware reciprocal off by an ulp
either way."""
import numpy as np
import pytest


def _multipliers(scale, d):
    r = np.float32(1) / np.float32(d)
    for rcp in (np.nextafter(r, np.float32(0)), r, np.nextafter(r, np.float32(2))):
        yield int(np.float32(np.float32(scale) * rcp)) + 1


@pytest.mark.parametrize("side", range(5, 65))
def test_tile_rows(side):
    ids = np.arange(4096, dtype=np.uint64)
    for m in _multipliers(262144.25, side):
        assert m == (1 << 18) // side + 1
        assert 4095 * m < 2**32 and ((ids * np.uint64(m)) >> np.uint64(18) == ids // np.uint64(side)).all()


@pytest.mark.parametrize("colours", range(1, 9))
def test_palette_indices(colours):
    ids = np.arange(4096, dtype=np.uint64)
    for m in _multipliers(65535.5, colours):
        assert m == 65535 // colours + 1 and m < 1 << 24
        assert ((ids * np.uint64(m)) >> np.uint64(16) == ids // np.uint64(colours)).all()
