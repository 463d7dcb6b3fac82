"""The tile sweep (records of a 4 x 4 quadrant broadcast between lanes, halo values
that no voxel uses not read) where it can go wrong: one-plane and one-column
last tiles, tiles deeper than the records staged at once, 8 x 8 tiles (four
quadrants, x3 values from memory), columns that carry planes from tile to tile,
blocks of solid that end stencils at every offset, both stencil rules and Maxwell
walls. Against the oracle, whose sums run in another order: 8 iterations of sums of
a few hundred terms stay within 8 x 300 x 2^-53, below 1e-11 relative to the
field's largest value."""
import numpy as np
import pytest

from oracle.oracle import OracleSolver
from paper_1712_01132_amd import poredvm

pytestmark = pytest.mark.gpu


def _mask(shape, seed):
    rng = np.random.default_rng(seed)
    m = np.zeros(shape, np.uint8)
    for _ in range(max(1, m.size // (60 if m.ndim == 3 else 20))):
        at = [rng.integers(0, n) for n in shape]
        m[tuple(slice(a, a + rng.integers(1, 6)) for a in at)] = 1
    m[(0,) * (len(shape) - 1)] = 0  # a free row along x1
    return m


@pytest.mark.parametrize("shape,tile,schedule", [
    ((5, 6, 9), (4, 4, 4), "queue"), ((13, 9, 17), (4, 4, 4), "columns"), ((9, 5, 6), (4, 4, 1), "columns"),
    ((21, 7, 10), (4, 4, 21), "queue"), ((19, 13, 10), (3, 4, 9), "diagonals"), ((10, 17, 9), (8, 8, 4), "queue"),
    ((11, 9, 18), (8, 8, 8), "diagonals"), ((9, 25), (4, 4), "queue"), ((35, 18), (8, 8), "queue"),
    ((17, 9), (8, 8), "diagonals"),
])
@pytest.mark.parametrize("kw", [dict(), dict(stencil_rule=0), dict(accommodation=0.7)])
def test_matches_the_oracle(shape, tile, schedule, kw):
    m = _mask(shape, sum(shape))
    nv = [6, 8, 6][:len(shape)]
    o = OracleSolver(m, nv, 0.6, threads=8, **kw)
    s = poredvm.Solver(m, nv, 0.6, tile=tile, schedule=schedule, grid=o.grid, **kw)
    assert s.schedule == schedule
    o.iterate(8)
    s.iterate(8)
    for a, b in zip(s.moments()[:2], o.moments()[:2]):
        assert np.abs(a - b).max() <= 1e-11 * np.abs(b).max()
    s.close()
