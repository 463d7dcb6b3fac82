"""Rows of nearly 1 GiB, the longest that the row pipeline takes, with tiles one or two
voxels wide: what the 4 x 4 kernel computes for the columns past a tile must be
dropped, at the start of a row and at its end. Against 4 x 4 tiles, bit for bit."""
import numpy as np
import pytest

from paper_1712_01132_amd import poredvm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [[1, 2], [2, 2]])
@pytest.mark.parametrize("alpha", [1.0, 0.8])
def test_narrow_tiles_on_the_longest_row(tile, alpha):
    n1 = 32766  # x 64 x 64 velocities in FP64 (32 KiB a voxel)
    mask = np.zeros((2, n1), np.uint8)
    mask[0, 5::97] = 1
    out = []
    for t in (tile, [4, 4]):
        s = poredvm.Solver(mask, [64, 64], 0.7, schedule="rows", tile=t, accommodation=alpha)
        s.iterate(2)
        out.append(s.moments(diagnostics=False))
        s.close()
    for x, y in zip(*out):
        assert np.array_equal(x, y)
