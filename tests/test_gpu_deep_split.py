"""The M2L's deep part has a launch of its own from 32 plane-wave tiles; the Hankel and FP32 forms, whose
tiles are smaller and slower, split whenever their tiles fill more than one level."""
import numpy as np
import pytest
import torch

import paper_2507_21913_amd as F
from oracle import direct as D

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,form,launches", [(2000, None, 1), (2000, "vector", 2), (2000, "mfma", 2),
                                             (2000, "fp32", 2), (100_000, None, 2)])
def test_m2l_launches(n, form, launches):
    rng = np.random.default_rng(n)
    x, y, q = (torch.as_tensor(v, device=DEV) for v in (rng.uniform(0, 1, n), rng.uniform(0.001, 1, n),
                                                        rng.standard_normal(n)))
    plan = F.HalfPlaneFMM(x, y, 1.0, p=20, leaf_size=20, m2l_fp32=form == "fp32",
                          m2l_form=form if form in ("vector", "mfma") else None)
    plan(q)
    F.fmmhp_plan_set_timing(plan._plan, 1)
    phi = plan(q).cpu().numpy()
    _, count = F.fmmhp_plan_m2l_kernel_times(plan._plan)
    F.fmmhp_plan_set_timing(plan._plan, 0)
    plan.close()
    assert count == launches
    if n <= 2000:
        ref = D.potential(x.cpu().numpy(), y.cpu().numpy(), q.cpu().numpy(), 1.0)
        assert D.rel_l2(phi, ref) < (1e-6 if form == "fp32" else 1e-10)
