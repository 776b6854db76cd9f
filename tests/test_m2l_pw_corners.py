"""The plane-wave quadratures where the expansions are at their worst: charges and targets on the edges and in
the corners of their boxes (the tables' own err is a root mean square over the boxes).

CPU: log potential of a unit charge at every offset of the east and west lists, p-term expansion with the
integrals (j-1)!/zeta^j and with the quadrature's sums, in extended precision.  The quadrature's error
stays below a tenth of the truncation's up to p = 30, a quarter at p = 35, and at p = 40, where the
truncation is 1.3e-15, below 1e-14: a rounding (2.2e-16) in each of the 41 coefficients.

GPU: unit charges in the corners of boxes, plane waves against the Hankel rows.  A charge reaches a far
target through one V pair: the error measured on the CPU over 2 pi, and a rounding in each coefficient
of both forms.
"""
import math
import os
import re

import numpy as np
import pytest

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_21913_amd", "csrc",
                      "pw_nodes.hpp")
BOUND = {5: 0.1, 10: 0.1, 15: 0.1, 20: 0.1, 25: 0.1, 30: 0.1, 35: 0.25, 40: None}
LD, CLD = np.longdouble, np.clongdouble


def _table(name):
    m = re.search(r"\b%s\[(\d+)\] = \{(.*?)\};" % name, open(HEADER).read(), re.S)
    return np.array([float(t) for t in m.group(2).replace("\n", " ").split(",")], dtype=LD)


def _worst(p):
    """Largest error of the quadrature and of the p-term expansion over pairs of points."""
    mu, om = _table(f"kPwMu{p}"), _table(f"kPwOm{p}")
    zs = np.array([2 * (dx + 1j * dy) for dx in (2, 3) for dy in range(-3, 4)], dtype=CLD)
    fact = [LD(1)]
    for k in range(1, 2 * p + 1):
        fact.append(fact[-1] * k)
    exact = np.zeros((2 * p + 1, zs.size), CLD)
    quad = np.zeros_like(exact)
    for i, z in enumerate(zs):
        t = om * np.exp(-mu * z)
        for j in range(1, 2 * p + 1):
            quad[j, i] = t.sum()
            exact[j, i] = fact[j - 1] / z ** j
            t = t * mu
    rng = np.random.default_rng(1)
    t, side = rng.uniform(-1, 1, 12), rng.integers(0, 4, 12)
    pts = [1 + 1j, 1 - 1j, -1 + 1j, -1 - 1j] + list(np.choose(side, [1 + 1j * t, -1 + 1j * t, t + 1j, t - 1j]))
    eq = et = 0.0
    for a in pts:
        ca = np.array([CLD(-a) ** k / fact[k] for k in range(p + 1)])
        for b in pts:
            c = np.convolve(ca, np.array([CLD(b) ** k / fact[k] for k in range(p + 1)]))
            eq = max(eq, float(np.abs(c @ (quad - exact)).max()))
            et = max(et, float(np.abs(c @ exact + np.log(1 - (CLD(b) - CLD(a)) / zs)).max()))
    return eq, et


@pytest.mark.parametrize("p", sorted(BOUND))
def test_error_in_the_corners(p):
    eq, et = _worst(p)
    print(f"p={p}: quadrature {eq:.1e}, truncation {et:.1e}")
    assert eq < (1e-14 if BOUND[p] is None else BOUND[p] * et)


torch = pytest.importorskip("torch")
import paper_2507_21913_amd as F  # noqa: E402

DEV = "cuda:0"


@pytest.mark.gpu
@pytest.mark.parametrize("p", [30, 35, 40])
def test_corner_charges_match_the_hankel_rows(p):
    # four points just inside the corners of each cell of a 16 x 8 grid: the root square is [0, 16] x [-8, 8]
    i, j = np.meshgrid(np.arange(16), np.arange(8), indexing="ij")
    d = 1e-7
    x = np.concatenate([(i + cx).ravel() for cx in (d, 1 - d) for _ in range(2)])
    y = np.concatenate([(j + cy).ravel() for _ in range(2) for cy in (d, 1 - d)])
    n = x.size
    src = np.random.default_rng(p).choice(n, 32, replace=False)
    q = np.zeros((32, n))
    q[np.arange(32), src] = 1.0
    out = []
    for form in (None, "vector"):
        plan = F.HalfPlaneFMM(torch.as_tensor(x, device=DEV), torch.as_tensor(y, device=DEV), 0.05, p=p, leaf_size=4,
                              m2l_form=form, bc="dirichlet")
        assert plan.info()["depth"] == 4 and plan.info()["m2l_pairs"][0] > 1000
        out.append(plan(torch.as_tensor(q, device=DEV)).cpu().numpy())
        plan.close()
    diff = float(np.abs(out[0] - out[1]).max())
    tol = _worst(p)[0] / (2 * math.pi) + 2 * (p + 1) * 2.2e-16
    print(f"p={p}: largest difference {diff:.1e}, tolerance {tol:.1e}")
    assert diff < tol
