"""A plan with more boxes than the list tables' launch has workgroups (65,536): a leaf size of one point, so
that the depth varies from leaf to leaf and every list is in use.

Tolerance: the truncation of the expansions, 10^(-p/2) at the separation of the lists.
"""
import numpy as np
import pytest
import torch

import paper_2507_21913_amd as F
from oracle import direct as D

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,p", [(150_001, 15)])
def test_more_boxes_than_workgroups(n, p):
    rng = np.random.default_rng(n)
    x, y, q = rng.uniform(0, 1, n), rng.uniform(0.001, 1, n), rng.standard_normal(n)
    plan = F.HalfPlaneFMM(*(torch.as_tensor(v, device=DEV) for v in (x, y)), 1.0 + 0.5j, p=p, leaf_size=1)
    info = plan.info()
    assert info["nbox"] > 2 * 65536 and min(info["list_len"]) > 0
    got = plan(torch.as_tensor(q, device=DEV)).cpu().numpy()
    plan.close()
    t = rng.choice(n, 64, replace=False)
    ref = D.potential(x, y, q, 1.0 + 0.5j, xt=x[t], yt=y[t])
    assert D.rel_l2(got[t], ref) < 10 ** (-p / 2)
