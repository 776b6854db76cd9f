"""The X list's rows without reaction terms, by slots: sixteen lanes a box (fewer than 16,384 X boxes) and
four, one and two vectors at a time, image rows with either sign, dipoles, against the oracle's direct
sums.  Points along a curve that comes down to the boundary; every tenth cluster of it is dense.

Tolerance: the truncation of the expansions, 10^(-p/2) at the separation of the lists, and not below 1e-12
(the near field's table logarithm).
"""
import numpy as np
import pytest
import torch

import paper_2507_21913_amd as F
from oracle import direct as D

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def _curve(n, seed):
    rng = np.random.default_rng(seed)
    t = np.where(rng.random(n) < 0.5, rng.random(n), rng.integers(0, 10, n) / 10 + 0.002 * rng.random(n))
    x = t + 1e-5 * rng.random(n)
    y = 0.3 * np.abs(np.sin(2 * np.pi * t)) + 1e-5 * rng.random(n) + 1e-6
    return x, y


def _x_boxes(plan):
    t = plan.export_tree()
    xo, xe = t["X_off"], t["X_ent"]
    return int((np.diff(xo) > 0).sum()), int((xe & 1).sum())


@pytest.mark.parametrize("n,p,bc,many", [(6000, 5, "neumann", False), (6000, 10, "robin", False),
                                         (6000, 15, "dirichlet", False), (6000, 20, "neumann", False),
                                         (6000, 40, "robin", False), (700_001, 10, "neumann", True),
                                         (700_001, 30, "neumann", True)])
def test_p2l_slots(n, p, bc, many):
    x, y = _curve(n, n + p)
    rng = np.random.default_rng(p)
    nv = 3 if many else 11
    q = rng.standard_normal((nv, n))
    plan = F.HalfPlaneFMM(_t(x), _t(y), 1.0 + 0.5j, p=p, leaf_size=20, bc=bc)
    nx, nimg = _x_boxes(plan)
    print(f"n={n} p={p} {bc}: {nx} X boxes, {nimg} image entries", flush=True)
    assert nimg > 0 and (nx >= 16384) == many
    phi = plan(_t(q)).cpu().numpy()
    for v in (0, nv - 1):
        assert np.array_equal(phi[v], plan(_t(q[v])).cpu().numpy())
    th = rng.uniform(0, 2 * np.pi, n)
    dl = plan.double_layer(_t(q[1]), _t(np.cos(th)), _t(np.sin(th))).cpu().numpy()
    plan.close()
    tol = max(10.0 ** (-p / 2), 1e-12)
    idx = rng.choice(n, 24 if many else 200, replace=False)
    ref = D.potential(x, y, q[0], 1.0 + 0.5j, xt=x[idx], yt=y[idx], bc=bc, workers=8)
    err = D.rel_l2(phi[0][idx], ref)
    ref = D.double_layer(x, y, np.cos(th), np.sin(th), q[1], 1.0 + 0.5j, xt=x[idx], yt=y[idx], bc=bc, workers=8)
    errd = D.rel_l2(dl[idx], ref)
    print(f"  potential {err:.1e}, double layer {errd:.1e}, tolerance {tol:.0e}", flush=True)
    assert err < tol and errd < 10 * tol
