"""The start distribution (16-byte chunks of slots, several voxels per thread) and
the diagnostics (octants of a velocity together) where they can go wrong: fewer
voxels than threads take at once, several rounds with a remainder, octants of
fewer slots than a chunk row, 2D and 3D. The first iteration reads the start
distribution through the images at every outer face, and the diagnostics sum the
distribution that it leaves. Against the oracle, whose sums run in another order:
FP64 sums of a few hundred terms stay within 300 x 2^-53 per pass, below 1e-12
relative to the field's scale; FP32 stores h to 2^-24, a few roundings per value,
below 1e-5."""
import numpy as np
import pytest

from oracle.oracle import OracleSolver
from paper_1712_01132_amd import poredvm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,nv", [((5, 3), [8, 8]), ((37, 23), [6, 10]), ((299, 301), [8, 8]), ((130, 64), [24, 24]),
                                      ((9, 11, 20), [4, 6, 4]), ((40, 33, 50), [8, 8, 8])])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_first_iteration_from_a_given_state(shape, nv, precision):
    rng = np.random.default_rng(sum(shape))
    m = (rng.random(shape) < 0.3).astype(np.uint8)
    m[(0,) * (len(shape) - 1)] = 0
    n1 = shape[-1]
    rho = np.where(m, 0, 0.5 - (np.arange(n1) + 0.5) / n1 + 0.05 * rng.standard_normal(shape))
    u = np.where(m, 0, 0.05 * rng.standard_normal((len(shape),) + shape))
    o = OracleSolver(m, nv, 0.6, threads=8)
    s = poredvm.Solver(m, nv, 0.6, precision=precision, grid=o.grid)
    o.set_initial(rho, u)
    s.set_initial(rho, u)
    o.iterate(1)
    s.iterate(1)
    for a, b in zip(s.moments(), o.moments()):
        scale = max(np.abs(b).max(), 0.1)
        assert np.abs(a - b).max() <= (1e-12 if precision == "fp64" else 1e-5) * scale
