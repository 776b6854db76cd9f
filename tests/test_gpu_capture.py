"""Calls of several charge vectors recorded into a graph of the caller's, on a plan that has only served
single vectors: nothing is allocated, the passes are as wide as the plan's present workspace, and every
replay, between the program's own eager work, gives the single vectors' results bitwise, also after an
eager call has grown the workspace.
"""
import threading

import numpy as np
import pytest
import torch

import paper_2507_21913_amd as F

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _plan(seed, n=4000, **kw):
    rng = np.random.default_rng(seed)
    x, y = rng.uniform(0, 1, n), rng.uniform(0.001, 1, n)
    plan = F.HalfPlaneFMM(torch.as_tensor(x, device=DEV), torch.as_tensor(y, device=DEV), 1.0 + 0.5j, p=15, leaf_size=20)
    return plan, rng


def _charges(rng, nvec, n, cplx):
    q = rng.standard_normal((nvec, n))
    if cplx:
        q = q + 1j * rng.standard_normal((nvec, n))
    return torch.as_tensor(q, device=DEV)


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("nvec", [2, 3, 7, 9])
def test_recorded_call_of_several_vectors(nvec, cplx):
    warm, rng = _plan(1)
    warm(_charges(rng, nvec, warm.n, cplx))  # loads the kernels
    warm.close()
    plan, rng = _plan(2)
    q, q2 = _charges(rng, nvec, plan.n, cplx), _charges(rng, nvec, plan.n, cplx)
    want = [torch.stack([plan(row) for row in c]) for c in (q, q2)]  # single vectors
    held = plan.info()["device_bytes"]
    out = torch.zeros((nvec, plan.n), dtype=torch.complex128, device=DEV)
    buf = q.clone()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        plan(buf, out=out)
    assert plan.info()["device_bytes"] == held
    for r in range(4):
        buf.copy_((q, q2)[r & 1])
        out.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[r & 1]), r
        if r == 1:
            assert torch.equal(plan(q), want[0])  # grows the workspace; the graph keeps the former one
            torch.cuda.synchronize()
    del g
    plan.close()


def test_growth_while_another_thread_records():
    """The first call of several vectors may come while another thread records a graph of its own."""
    warm, rng = _plan(1)
    warm(_charges(rng, 3, warm.n, False))
    plan, rng = _plan(3)
    q = _charges(rng, 3, plan.n, False)
    want = torch.stack([plan(row) for row in q])
    out = torch.zeros((3, plan.n), dtype=torch.complex128, device=DEV)
    torch.cuda.synchronize()
    res = []

    def work():
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                plan(q, out=out)
            res.append("ok")
        except Exception as e:  # noqa: BLE001 -- reported by the main thread
            res.append(e)

    a = torch.ones(8, device=DEV)
    g = torch.cuda.CUDAGraph()
    t = threading.Thread(target=work)
    with torch.cuda.graph(g):
        b = a * 2
        t.start()
        t.join()
    torch.cuda.synchronize()
    assert res == ["ok"]
    g.replay()
    torch.cuda.synchronize()
    assert torch.equal(out, want) and torch.equal(b, a * 2)
    plan.close()
    warm.close()
