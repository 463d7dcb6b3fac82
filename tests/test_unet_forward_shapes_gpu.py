"""The network's forward pass at sizes where its tiles are ragged: images narrower
than a tile, sides that are no multiple of one, deepest levels of one pixel (a
wrong border column or row of a convolution shows in the largest difference).
Against the float64 reference that rounds to bfloat16 at the same places; weights
and bounds are those of the forward test in test_warmstart_gpu.py (FP32 sums flip
about 2 % of the bfloat16 roundings by one step: 5e-3 of the output, 2e-2 of its
largest value at a single pixel)."""
import numpy as np
import pytest

from oracle import unet_oracle as U

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,B", [(8, 8, 5), (24, 16, 3), (16, 136, 1), (40, 72, 2), (264, 24, 1), (72, 40, 4), (8, 256, 2)])
def test_forward_matches_the_reference(n1, n2, B):
    from paper_1712_01132_amd import warmstart
    rng = np.random.default_rng(n1 + n2)
    solids = [(rng.random((n2, n1)) < 0.4).astype(np.uint8) for _ in range(B)]
    kns = [float(k) for k in np.exp(rng.uniform(np.log(0.05), np.log(20), B))]
    params = warmstart.init_params(3)
    params[-3:] = [0.1, -0.2, 0.05]
    net = warmstart.Net(n1, n2, batch_max=B, dataset_max=B)
    net.set_params(params)
    for i in range(B):
        net.set_sample(i, solids[i], kns[i], np.zeros((n2, n1)), np.zeros((2, n2, n1)))
    out = net.forward(list(range(B)))
    net.close()
    ref = U.forward(params, U.make_input(solids, kns)).numpy()
    got = np.transpose(out[..., :3], (0, 3, 1, 2))
    assert np.all(out[..., 3] == 0)
    assert np.linalg.norm(got - ref) <= 5e-3 * np.linalg.norm(ref)
    assert np.abs(got - ref).max() <= 2e-2 * np.abs(ref).max()
