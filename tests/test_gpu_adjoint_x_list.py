"""The adjoint (three charge vectors a pass, potentials and gradients) on a set with X and W lists, upper and
image, against the oracle's direct gradients.  Tolerance: the truncation of the expansions at p = 30,
10^(-p/2) at the separation of the lists, enlarged to 1e-11 for the cancellation in the gradients' sums.
"""
import numpy as np
import pytest
import torch

import paper_2507_21913_amd as F
from oracle import grad as G

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


@pytest.mark.parametrize("Z", [1.0, 1.0 + 0.5j])
@pytest.mark.parametrize("p", [20, 30])
def test_adjoint_with_x_and_w_lists(Z, p):
    rng = np.random.default_rng(5)
    n = 1600
    x = np.concatenate([rng.random(800), 0.3 + 0.02 * rng.random(400), 0.7 + 0.02 * rng.random(400)])
    y = np.concatenate([rng.random(800), 1e-3 + 0.02 * rng.random(400), 0.5 + 0.02 * rng.random(400)])
    q = rng.standard_normal(n)
    g = rng.standard_normal(n) + 1j * rng.standard_normal(n)
    plan = F.HalfPlaneFMM(_t(x), _t(y), Z, p=p, leaf_size=12)
    t = plan.export_tree()
    assert (t["X_ent"] & 1).any() and not (t["X_ent"] & 1).all() and (t["W_ent"] & 1).any()
    b = plan.backward(_t(q), _t(g))
    plan.close()
    r = G.direct_gradients(x, y, q, Z, g)
    tol = max(10.0 ** (-p / 2), 1e-11)
    for k in ("q", "x", "y"):
        e = np.linalg.norm(b[k].cpu().numpy() - r["grad_" + k]) / np.linalg.norm(r["grad_" + k])
        print(f"Z={Z} p={p} grad_{k}: {e:.1e}", flush=True)
        assert e < 10 * tol, k
