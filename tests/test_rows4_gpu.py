"""The 4x4 row pipeline (records broadcast between lanes, importer wavefronts,
solid tiles that do not wait) where it can go wrong: ragged last tiles along
x1 and x2, bands that end on and next to a tile row, thin tiles, images a few
voxels wide, and geometries whose tiles are partly or wholly solid. Every
schedule runs the same arithmetic, so the iterates must equal those of the tile
diagonals bit for bit; FP64 is also held against the oracle, whose sums run
in another order: 20 iterations of sums of a few hundred terms stay within
20 x 300 x 2^-53, below 1e-11 relative to the field's largest value."""
import numpy as np
import pytest

from paper_1712_01132_amd import geometry, poredvm

pytestmark = pytest.mark.gpu


def _mask(n1, n2, seed):
    """Blocks of solid several tiles wide (whole tiles solid, and tiles cut at
    every offset), with one free row so that x1 percolates."""
    rng = np.random.default_rng(seed)
    m = np.zeros((n2, n1), np.uint8)
    for _ in range(max(1, n1 * n2 // 150)):
        x, y = rng.integers(0, n1), rng.integers(0, n2)
        m[y:y + rng.integers(1, 14), x:x + rng.integers(1, 14)] = 1
    m[n2 // 2, :] = 0
    return m


def _run(mask, schedule, iters, **kw):
    s = poredvm.Solver(mask, kw.pop("nv", [8, 8]), 0.7, schedule=schedule, **kw)
    st = s.iterate(iters)
    f = s.moments()
    blob = s.get_state()
    used = s.schedule
    s.close()
    return st, f, blob, used


@pytest.mark.parametrize("n1,n2", [(2, 2), (3, 33), (5, 31), (8, 64), (9, 65), (33, 3), (40, 95), (67, 129), (130, 36)])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_equals_the_tile_diagonals(n1, n2, precision):
    mask = _mask(n1, n2, n1 * 1000 + n2)
    a = _run(mask, "rows", 20, tile=[4, 4], precision=precision)
    b = _run(mask, "diagonals", 20, tile=[4, 4], precision=precision)
    assert a[3].startswith("rows") and b[3] == "diagonals"
    assert a[0]["r"] == b[0]["r"] and a[0]["k"] == b[0]["k"]
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y)
    assert a[2] == b[2]


@pytest.mark.parametrize("tile", [[1, 1], [2, 3], [3, 1], [4, 2]])
@pytest.mark.parametrize("kw", [dict(), dict(tau_feedback=True), dict(tau_feedback=True, prandtl=2 / 3),
                                dict(lateral="periodic")])
def test_thin_tiles_and_models(tile, kw):
    mask = _mask(37, 50, 5)
    for precision in ("fp64", "fp32"):
        a = _run(mask, "rows", 12, tile=tile, precision=precision, nv=[8, 12], **kw)
        b = _run(mask, "diagonals", 12, tile=[4, 4], precision=precision, nv=[8, 12], **kw)
        for x, y in zip(a[1], b[1]):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("nv", [[8, 8], [16, 18], [24, 24]])
def test_agent_scope_protocol_and_velocity_groups(nv):
    """Partial last 64-velocity groups, several groups per octant; both
    publication protocols."""
    mask = _mask(45, 75, 9)
    b = _run(mask, "diagonals", 8, tile=[4, 4], nv=nv)
    for schedule in ("rows", "rows-agent"):
        a = _run(mask, schedule, 8, tile=[4, 4], nv=nv)
        for x, y in zip(a[1], b[1]):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("n1,n2", [(6, 34), (67, 129)])
def test_matches_the_oracle(n1, n2):
    from oracle.oracle import OracleSolver
    mask = _mask(n1, n2, 3)
    o = OracleSolver(mask, [8, 8], 0.7, threads=8)
    o.iterate(20)
    ref = o.moments()
    got = _run(mask, "rows", 20, tile=[4, 4], grid=o.grid)[1]
    for x, y in zip(got[:2], ref[:2]):
        assert np.max(np.abs(x - y)) <= 1e-11 * np.max(np.abs(y))


def test_channel_without_solid_tiles():
    mask = geometry.plane_channel(72, 70)
    a = _run(mask, "rows", 20, tile=[4, 4])
    b = _run(mask, "diagonals", 20, tile=[8, 8])
    for x, y in zip(a[1], b[1]):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("n1,n2,tile", [(2, 3, [4, 4]), (9, 65, [4, 4]), (40, 95, [4, 4]), (33, 37, [3, 1]), (131, 66, [2, 3])])
@pytest.mark.parametrize("kw", [dict(), dict(tau_feedback=True), dict(tau_feedback=True, prandtl=2 / 3),
                                dict(lateral="periodic")])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_maxwell_walls_equal_the_tile_diagonals(n1, n2, tile, kw, precision):
    """Tiles with walls along one axis, both or none, ragged and thin tiles."""
    mask = _mask(n1, n2, n1 + n2)
    for schedule in ("rows", "rows-agent"):
        a = _run(mask, schedule, 12, tile=tile, precision=precision, nv=[8, 12], accommodation=0.7, **kw)
        b = _run(mask, "diagonals", 12, tile=[4, 4], precision=precision, nv=[8, 12], accommodation=0.7, **kw)
        for x, y in zip(a[1], b[1]):
            assert np.array_equal(x, y)
