"""Row pipelines with tiles one voxel high: a band's two halo rows then come from
two wavefronts of the band below, and the counter that one of them publishes
has to stand for the stores of both. Many bands, long rows, both publication
protocols and both kernels (4 x 4 and 8 x 8 edges, stencil rules 0 and 1); every
schedule runs the same arithmetic, so the iterates must equal those of the tile
diagonals bit for bit."""
import numpy as np
import pytest

from paper_1712_01132_amd import poredvm

pytestmark = pytest.mark.gpu


def _run(mask, schedule, iters=10, **kw):
    s = poredvm.Solver(mask, [8, 12], 0.7, schedule=schedule, **kw)
    st = s.iterate(iters)
    f = s.moments()
    s.close()
    return st["r"], st["k"], f


@pytest.mark.parametrize("tile", [[4, 1], [1, 1], [8, 1]])
@pytest.mark.parametrize("rule", [1, 0])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n1,n2", [(301, 9), (150, 101)])
def test_one_voxel_rows_equal_the_tile_diagonals(tile, rule, precision, n1, n2):
    rng = np.random.default_rng(n1 + n2)
    mask = (rng.random((n2, n1)) < 0.15).astype(np.uint8)
    mask[n2 // 2] = 0
    b = _run(mask, "diagonals", tile=[4, 4], stencil_rule=rule, precision=precision)
    for schedule in ("rows", "rows-agent"):
        a = _run(mask, schedule, tile=tile, stencil_rule=rule, precision=precision)
        assert a[:2] == b[:2]
        for x, y in zip(a[2], b[2]):
            assert np.array_equal(x, y)
