"""The network's gradients at sizes where their tiles
are ragged: images one patch wide and narrower, sides that are no multiple of a
32-pixel patch, batches that fill no block, deepest levels of 1 to 3 pixels.
Against the float64 reference that rounds to bfloat16 at the same places; the
bound is the one derived in test_warmstart_gpu.py (FP32 sums flip about 2 % of
the bfloat16 roundings by one step: 2e-2 of a layer's gradient)."""
import numpy as np
import pytest

from oracle import unet_oracle as U

pytestmark = pytest.mark.gpu


def _net(n1, n2, B, seed):
    from paper_1712_01132_amd import geometry, warmstart
    rng = np.random.default_rng(seed)
    solids = [(rng.random((n2, n1)) < 0.4).astype(np.uint8) for _ in range(B)]
    kns = [float(k) for k in np.exp(rng.uniform(np.log(0.05), np.log(20), B))]
    rhos = [rng.standard_normal((n2, n1)) * 0.2 for _ in range(B)]
    us = [rng.standard_normal((2, n2, n1)) * 0.01 for _ in range(B)]
    params = warmstart.init_params(seed)
    params[warmstart.weight_mask() == 0] = rng.standard_normal(int((~warmstart.weight_mask()).sum())) * 0.1
    net = warmstart.Net(n1, n2, batch_max=B, dataset_max=B)
    net.set_params(params)
    for i in range(B):
        net.set_sample(i, solids[i], kns[i], rhos[i], us[i])
    return net, params, solids, kns, rhos, us


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("n1,n2,B", [(8, 8, 5), (24, 16, 3), (16, 136, 1), (40, 72, 2), (264, 24, 1), (72, 40, 4)])
def test_shapes_match_the_reference(n1, n2, B):
    net, params, solids, kns, rhos, us = _net(n1, n2, B, n1 + n2)
    loss = net.train_step(list(range(B)), update=False)
    g = net.grads()
    net.close()
    targets, ws = zip(*[U.make_targets(s, r, u, k) for s, r, u, k in zip(solids, rhos, us, kns)])
    lref, gref = U.loss_and_grads(params, solids, kns, list(targets), list(ws))
    assert abs(loss - lref) <= 1e-3 * abs(lref)
    o = 0
    for cout, taps, cin in U.ARCH:
        nw = cout * taps * cin
        assert _rel(g[o:o + nw], gref[o:o + nw]) <= 2e-2
        assert _rel(g[o + nw:o + nw + cout], gref[o + nw:o + nw + cout]) <= 2e-2
        o += nw + cout
