"""Near-field records at the edges of their lane layout: leaves of 1 to 130 points (one to sixteen lane
groups of one to four targets, records cut at 64 targets, streams that end inside a step), with
coincident points, for the potential, eight vectors at once, the gradient, the double layer and the
adjoint, against the oracle's direct sums.

All points lie in the boxes of level 1, so every pair is a near-field pair.  Tolerance: the table
logarithm is good to 2.5e-13 per pair, absolute, in terms of order one: 1e-12 relative in the potential
of random charges; derivatives take a reciprocal instead (rounding only, enlarged by the nearest pair).
"""
import numpy as np
import pytest
import torch

import paper_2507_21913_amd as F
from oracle import direct as D
from oracle import grad as G

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def _off(a, b):
    """Relative l2 error; absolute where the exact value is zero (a single point has no d/dx)."""
    return np.linalg.norm(a - b) / (np.linalg.norm(b) or 1.0)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 130])
@pytest.mark.parametrize("Z", [1.0, 1.0 + 0.5j])
def test_one_leaf(n, Z):
    rng = np.random.default_rng(n)
    x, y = rng.uniform(0.4, 0.6, n), rng.uniform(0.01, 0.21, n)
    if n >= 8:
        x[3], y[3] = x[5], y[5]
    q = rng.standard_normal((8, n))
    plan = F.HalfPlaneFMM(_t(x), _t(y), Z, p=10, leaf_size=n)
    assert plan.info()["depth"] == 1
    phi = plan(_t(q)).cpu().numpy()
    for v in (0, 7):
        ref = D.potential(x, y, q[v], Z, workers=1)
        assert D.rel_l2(phi[v], ref) < 1e-12
        assert np.array_equal(phi[v], plan(_t(q[v])).cpu().numpy())
    f, gx, gy = (t.cpu().numpy() for t in plan.field(_t(q[0])))
    rx, ry = G.potential_gradient(x, y, q[0], Z)
    assert D.rel_l2(f, phi[0]) < 1e-13
    assert _off(gx, rx) < 1e-11 and _off(gy, ry) < 1e-11
    th = rng.uniform(0, 2 * np.pi, n)
    dl = plan.double_layer(_t(q[1]), _t(np.cos(th)), _t(np.sin(th))).cpu().numpy()
    ref = D.double_layer(x, y, np.cos(th), np.sin(th), q[1], Z, workers=1)
    assert _off(dl, ref) < 1e-11
    g = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    b = plan.backward(_t(q[0]), _t(g))
    r = G.direct_gradients(x, y, q[0], Z, g)
    for k in ("q", "x", "y"):
        assert _off(b[k].cpu().numpy(), r["grad_" + k]) < 1e-11, k
    assert abs(b["lambda"] - r["grad_Z"]) < 1e-10 * max(1.0, abs(r["grad_Z"]))
    plan.close()
