"""pdvm_iterate_noalloc at the limit of the library's static scratch."""
import numpy as np
import pytest

from paper_1712_01132_amd import poredvm

pytestmark = pytest.mark.gpu


def test_partials_that_do_not_fit_the_scratch():
    """A queue of one-voxel tiles whose done flags (128 chains x 8142 tiles x 4
    bytes) leave room in the 4 MiB for the partial sums of 128 blocks (16 voxels per
    wavefront) but not for those of the 256 the moments run with: the partials
    stay in the workspace."""
    m = np.zeros((23, 6, 59), np.uint8)
    m[12, 3, 40] = 1
    out = []
    for name in ("iterate", "iterate_noalloc"):
        s = poredvm.Solver(m, [16, 16, 32], 0.6, precision="fp32", schedule="queue", tile=[1, 1, 1])
        st = getattr(s, name)(2)
        out.append((st["k"], st["r"], s.moments()))
        s.close()
    assert out[0][:2] == out[1][:2]
    for x, y in zip(out[0][2], out[1][2]):
        assert np.array_equal(x, y)
