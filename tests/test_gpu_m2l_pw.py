"""The plane-wave M2L of upper sources (the default form): its quadrature tables against the integrals
they stand for (CPU), and on the GPU against the Hankel rows of the vector form
(FMMHP_FLAG_M2L_VECTOR), which compute the same sums exactly.

Tolerance: an entry of a table names the root mean square error err that the quadrature leaves in the
far field of a unit charge pair at a V offset.  With random charges both the far field and its error
grow like the square root of the sources, so the relative difference of two potentials is of the
order of err: 4 err, plus 1e-14 for the two orders of summation.

Sets: tiles of one parent and of a few, a uniform set whose levels hold 16 to 1024 parents (tiles filled
exactly and partly, cut at 63 source cells at other alignments), an adaptive band with missing children
and colleagues, and a forest whose tiles hold boxes of several instances.
"""
import math
import os
import re

import numpy as np
import pytest

ERR = {5: 1.1e-12, 10: 9.6e-13, 15: 8.8e-13, 20: 1.1e-13, 25: 5.5e-15, 30: 4.7e-16, 35: 9.1e-17, 40: 9.1e-17}
HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_21913_amd", "csrc",
                      "pw_nodes.hpp")


def _table(name):
    m = re.search(r"\b%s\[(\d+)\] = \{(.*?)\};" % name, open(HEADER).read(), re.S)
    v = np.array([float(t) for t in m.group(2).replace("\n", " ").split(",")])
    assert v.size == int(m.group(1))
    return v


@pytest.mark.parametrize("p", sorted(ERR))
def test_quadrature_reproduces_the_hankel_entries(p):
    """sum_k omega_k mu_k^(j-1) e^(-mu_k zeta) = (j-1)!/zeta^j at the fourteen offsets, each j = 1..2p
    weighed with the rms of its coefficient over points uniform in the two boxes."""
    mu, om = _table(f"kPwMu{p}"), _table(f"kPwOm{p}")

    def moment(n):  # mean of |b|^(2n) over [-1, 1]^2
        return sum(math.comb(n, k) / (2 * k + 1) / (2 * (n - k) + 1) for k in range(n + 1))

    total = 0.0
    for j in range(1, 2 * p + 1):
        s2 = sum(moment(n) * moment(j - n) / (math.factorial(n) * math.factorial(j - n)) ** 2
                 for n in range(max(0, j - p), min(p, j) + 1))
        for dx in (2, 3):
            for dy in range(-3, 4):
                z = 2.0 * complex(dx, dy)
                e = np.sum(om * mu ** (j - 1) * np.exp(-mu * z)) - math.factorial(j - 1) / z ** j
                total += s2 * abs(e) ** 2
    # 3e-15: float64 rounding of the sums above
    assert math.sqrt(total / 14) < ERR[p] + 3e-15


torch = pytest.importorskip("torch")
import paper_2507_21913_amd as F  # noqa: E402
from oracle import direct as D  # noqa: E402

DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


def _points(kind, rng):
    if kind == "one_tile":       # a handful of boxes
        return rng.uniform(0, 1, 60), rng.uniform(0.01, 1, 60)
    if kind == "uniform":
        return rng.uniform(0, 1, 20000), rng.uniform(0.001, 1, 20000)
    if kind == "narrow":         # a row of parents: few colleagues each, many parents per tile
        return rng.uniform(0, 64, 9000), rng.uniform(0.001, 0.6, 9000)
    n = 6000                     # "band": half the points near the axis and in a cluster
    x = np.concatenate([rng.uniform(0, 1, n // 2), 0.3 + 0.01 * rng.standard_normal(n // 4),
                        rng.uniform(0, 1, n - n // 2 - n // 4)])
    y = np.concatenate([rng.uniform(1e-3, 0.05, n // 2), 0.4 + 0.01 * rng.standard_normal(n // 4),
                        rng.uniform(1e-3, 1, n - n // 2 - n // 4)])
    return x, y


def _both(make, q):
    out = []
    for form in (None, "vector"):
        plan = make(form)
        out.append(plan(_t(q)).cpu().numpy())
        plan.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["one_tile", "uniform", "narrow", "band"])
@pytest.mark.parametrize("p", sorted(ERR))
def test_matches_the_hankel_rows(kind, p):
    rng = np.random.default_rng(p)
    x, y = _points(kind, rng)
    Z = 0.05 if kind == "narrow" else 1.0 + 0.5j
    q = rng.standard_normal(x.size)
    pw, vec = _both(lambda f: F.HalfPlaneFMM(_t(x), _t(y), Z, p=p, leaf_size=5 if kind == "uniform" else 12,
                                             m2l_form=f), q)
    err = D.rel_l2(pw, vec)
    print(f"{kind} p={p}: plane waves vs Hankel rows rel-l2 {err:.2e}", flush=True)
    assert err < 4 * ERR[p] + 1e-14


@pytest.mark.gpu
def test_forest_and_vectors():
    """Tiles across instances, eight vectors and one, dipoles (w_0 = 0) and gradients."""
    rng = np.random.default_rng(8)
    sizes = [700, 30, 2500, 1, 400]
    off = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    x, y = rng.uniform(0, 1, off[-1]), rng.uniform(0.01, 1.01, off[-1])
    q = rng.standard_normal((9, off[-1]))
    Zs = [0.5, 3.0, 1.0 + 0.5j, 2.0, 8.0]
    pw, vec = _both(lambda f: F.HalfPlaneFMM.batched(_t(x), _t(y), off, Zs, p=20, leaf_size=10, m2l_form=f), q)
    assert D.rel_l2(pw, vec) < 4 * ERR[20] + 1e-14
    th = rng.uniform(0, 2 * np.pi, off[-1])
    res = []
    for form in (None, "vector"):
        plan = F.HalfPlaneFMM(_t(x), _t(y), 1.0, p=20, leaf_size=10, m2l_form=form)
        res.append((plan.double_layer(_t(q[0]), _t(np.cos(th)), _t(np.sin(th))).cpu().numpy(),
                    plan.field(_t(q[0]))[1].cpu().numpy()))
        plan.close()
    # one derivative more: a factor 2 (p + 1) at most between the coefficients of f and of f'
    for a, b in zip(*res):
        assert D.rel_l2(a, b) < 42 * 4 * ERR[20] + 1e-13
