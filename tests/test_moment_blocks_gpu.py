"""The moment kernel where a batch has more logical blocks than the chip needs, so
that a block does several of them (up to 8, by the voxels each has): every sum
has to be the one that the problem has alone, where each logical block is a
block. Problems of a handful of fluid voxels, of one logical block's share more
or less, and of more than 16384; the kernel's slot layouts (paired slots, two
voxels per wavefront with odd counts, one voxel) in 2D and 3D."""
import numpy as np
import pytest

from paper_1712_01132_amd import poredvm

pytestmark = pytest.mark.gpu


def _mask(shape, seed):
    m = (np.random.default_rng(seed).random(shape) < 0.25).astype(np.uint8)
    m[(shape[0] // 2,) * (len(shape) - 1)] = 0
    return m


SHAPES2 = [(2, 3), (3, 3), (7, 11), (17, 13), (56, 49)] + [(45, 40 + 3 * i) for i in range(12)] + [(150, 160)]
SHAPES3 = [(2, 3, 4), (5, 6, 7)] + [(14, 14, 12 + i) for i in range(12)] + [(28, 30, 31)]


@pytest.mark.parametrize("shapes,nv,precision", [(SHAPES2, [8, 8], "fp64"), (SHAPES2, [8, 8], "fp32"), (SHAPES2, [6, 6], "fp64"),
                                                 (SHAPES2, [24, 24], "fp32"), (SHAPES3, [6, 6, 6], "fp64"),
                                                 (SHAPES3, [8, 8, 8], "fp32")])
def test_sums_in_a_large_batch_are_those_of_the_problems_alone(shapes, nv, precision):
    probs = [(_mask(s, i), 0.3 + 0.1 * i) for i, s in enumerate(shapes)]
    fluid = [int((m == 0).sum()) for m, _ in probs]
    assert sum(max(min((f + 63) // 64, 1024), min((f + 7) // 8, 256)) for f in fluid) > 2048  # else nothing is folded
    b = poredvm.Batch(probs, nv, precision=precision)
    rb = b.iterate(5)
    for i, (m, kn) in enumerate(probs):
        s = poredvm.Solver(m, nv, kn, precision=precision)
        rs = s.iterate(5)
        assert (rs["k"], rs["r"], rs["Gp"]) == (rb[i]["k"], rb[i]["r"], rb[i]["Gp"])
        for x, y in zip(s.moments(diagnostics=False), b.moments(i)):
            assert np.array_equal(x, y)
        s.close()
    b.close()
