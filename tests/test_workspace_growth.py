"""Growth of a plan's workspaces where device memory is short: the host code of arena.hpp and workspace.hpp
compiled for the CPU against a hipMalloc that fails on demand (CPU), and on the GPU through the allocation
hook FMMHP_TEST_FAIL_ALLOC ("k": the k-th array of a plan fails, "k+": every one from it on).

A workspace that could not grow keeps its pointers and width, nothing is taken for the failed attempt,
narrower widths are tried, and a width that failed is not tried again.  On the GPU a call of several
vectors that had to go narrower gives the vectors' results of single calls bitwise.
"""
import os
import re
import subprocess
import textwrap

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_21913_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

DRIVER = textwrap.dedent(r"""
    #include <assert.h>
    #include <stdarg.h>
    #include <stdio.h>
    #include <string.h>
    #include <map>
    #include "workspace.hpp"
    using namespace fmmhp;

    static std::map<char *, size_t> live;   // device allocations: address -> bytes
    static char *next_at = (char *)0x10000000000;
    static size_t largest = (size_t)-1;     // larger requests fail
    static int calls = 0;
    extern "C" hipError_t hipMalloc(void **p, size_t n) {
        ++calls;
        if (n > largest) return hipErrorOutOfMemory;
        *p = next_at;
        live[next_at] = n;
        next_at += (n + 4095) / 4096 * 4096 + 4096;
        return hipSuccess;
    }
    extern "C" hipError_t hipFree(void *p) { live.erase((char *)p); return hipSuccess; }
    extern "C" hipError_t hipGetLastError() { return hipSuccess; }
    extern "C" const char *hipGetErrorString(hipError_t) { return "out of memory"; }
    namespace fmmhp { void set_error(const char *, ...) {} }

    static size_t total() { size_t t = 0; for (auto &a : live) t += a.second; return t; }
    static void inside(const void *p, size_t n) {  // [p, p + n) lies in one live allocation
        for (auto &a : live)
            if ((char *)p >= a.first && (char *)p + n <= a.first + a.second) return;
        printf("array outside the live allocations\n");
        exit(1);
    }
    static void check_ws(const Tree &T, const Sched &S) {
        const VecWs &w = S.ws;
        const size_t nv = w.cap, P1 = S.PB + 1;
        inside(w.W, nv * P1 * T.nbox * 16);
        inside(w.Lam, nv * S.nloc * P1 * T.nbox * 16);
        inside(w.qs, nv * T.n * 8);
        inside(w.near, nv * T.n * 16);
        inside(w.red, nv * S.n_rch * 16);
        inside(w.rank1, nv * T.n_inst * 16);
        if (S.m2l_fp32) inside(w.Wf, nv * T.nbox * m2l32_kp(S.PB) * 4);
        if (S.near_walk >= 3) inside(w.part, nv * S.sym_npart * 8);
    }
    struct Plan {
        Arena A; Tree T; Sched S;
        Plan(int form) {
            live.clear(); largest = (size_t)-1; calls = 0;
            T.n = 200003; T.nbox = 20001; T.n_inst = 3;
            S.PB = 20; S.nloc = 1 + (form & 1); S.n_rch = 99; S.m2l_fp32 = form & 2;
            if (form & 4) { S.sym_ok = true; S.near_walk = 4; S.sym_npart = 777777; }
            assert(ensure_vec_ws(A, T, S, 1) == FMMHP_OK && S.ws.cap == 1);
            check_ws(T, S);
        }
        size_t bytes(int nv) { return vec_ws_layout(T, S, nv, nullptr, nullptr); }
    };

    int main() {
        for (int form = 0; form < 8; ++form)
            for (int nvec = 1; nvec <= 17; ++nvec) {
                const int want = nvec >= 8 ? 8 : nvec >= 4 ? 4 : nvec >= 2 ? 2 : 1;
                for (int fit = 1; fit <= want; fit *= 2) {  // widths above fit do not fit
                    Plan p(form);
                    const VecWs before = p.S.ws;
                    const size_t t0 = total();
                    largest = fit == 1 ? 0 : p.bytes(fit);
                    const int c0 = calls;
                    assert(ensure_eval_ws(p.A, p.T, p.S, nvec) == FMMHP_OK);
                    assert(p.S.ws.cap == fit);
                    check_ws(p.T, p.S);
                    if (fit == 1) assert(memcmp(&before, &p.S.ws, sizeof before) == 0 && total() == t0);
                    else assert(total() == t0 + p.bytes(fit));
                    const size_t t1 = total(), b1 = p.A.bytes;
                    assert((size_t)p.A.held == t1);  // fmmhp_plan_stats.device_bytes
                    const int c1 = calls;
                    for (int r = 0; r < 5; ++r) assert(ensure_eval_ws(p.A, p.T, p.S, nvec) == FMMHP_OK);
                    assert(calls == c1 && total() == t1 && (size_t)p.A.bytes == b1);
                    largest = 0;  // the three-vector workspace of the adjoint: refused, nothing changed
                    const VecWs w1 = p.S.ws;
                    const fmmhp_status st = ensure_vec_ws(p.A, p.T, p.S, 9);
                    assert(st == FMMHP_ENOMEM && memcmp(&w1, &p.S.ws, sizeof w1) == 0 && total() == t1);
                    p.A.release();
                    assert(live.empty() && p.A.bytes == 0 && p.A.held == 0 && c1 >= c0);
                }
                for (int k = 1; k <= 4; ++k) {  // one failing call: what is there afterwards is whole
                    Plan p(form);
                    setenv("FMMHP_TEST_FAIL_ALLOC", std::to_string(p.A.tries + k).c_str(), 1);
                    assert(ensure_eval_ws(p.A, p.T, p.S, nvec) == FMMHP_OK);
                    unsetenv("FMMHP_TEST_FAIL_ALLOC");
                    check_ws(p.T, p.S);
                    assert(p.S.ws.cap == (k > 1 || want == 1 ? want : want / 2));
                }
            }
        for (int g = 1; g <= 4; ++g) {  // complex charges
            Plan p(0);
            const size_t t0 = total(), one = 48 * p.T.n;
            largest = 0;
            auto grow = [&](int w) { return ensure_split(p.A, p.T, p.S, w); };
            for (int r = 0; r < 3; ++r) {
                assert(widen(g, p.S.ccap, p.S.ccap_limit, grow) == FMMHP_ENOMEM);
                assert(!p.S.cq && !p.S.cphi && p.S.ccap == 0 && total() == t0);
            }
            largest = one + 4096;
            assert(widen(g, p.S.ccap, p.S.ccap_limit, grow) == FMMHP_OK && p.S.ccap == 1);
            inside(p.S.cq, 16 * p.T.n);
            inside(p.S.cphi, 32 * p.T.n);
            const size_t t1 = total();
            assert(widen(4, p.S.ccap, p.S.ccap_limit, grow) == FMMHP_OK && p.S.ccap == 1 && total() == t1);
        }
        {  // adjoint
            Plan p(0);
            const size_t t0 = total();
            largest = 0;
            assert(ensure_bwd(p.A, p.T, p.S) == FMMHP_ENOMEM && !p.S.bw.ready && !p.S.bw.red && total() == t0);
            largest = (size_t)-1;
            assert(ensure_bwd(p.A, p.T, p.S) == FMMHP_OK && p.S.bw.ready);
            for (cplx *c : {p.S.bw.phi3, p.S.bw.gx3, p.S.bw.gy3, p.S.bw.near_gx, p.S.bw.near_gy}) inside(c, 48 * p.T.n);
            inside(p.S.bw.red, 16 * (p.S.n_rch + p.T.n_inst));
        }
        printf("GROWTH_OK\n");
        return 0;
    }
""")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc is needed")
def test_growth_is_all_or_nothing(tmp_path):
    src, exe = tmp_path / "grow.hip", tmp_path / "grow"
    src.write_text(DRIVER)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    env = {k: v for k, v in os.environ.items() if k != "FMMHP_TEST_FAIL_ALLOC"}
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, env=env)
    assert r.returncode == 0 and "GROWTH_OK" in r.stdout, r.stdout + r.stderr


torch = pytest.importorskip("torch")
import paper_2507_21913_amd as F  # noqa: E402

DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


@pytest.fixture
def alloc_hook():
    yield lambda v: os.environ.__setitem__("FMMHP_TEST_FAIL_ALLOC", v)
    os.environ.pop("FMMHP_TEST_FAIL_ALLOC", None)


# no array of the call fits; or only its first (the widest pass) does not
@pytest.mark.gpu
@pytest.mark.parametrize("nvec", [2, 3, 7, 8, 17])
@pytest.mark.parametrize("fail", ["1+", "first"])
def test_short_memory_takes_narrower_passes(nvec, fail, alloc_hook):
    rng = np.random.default_rng(nvec)
    n = 5000
    x, y = _t(rng.uniform(0, 1, n)), _t(rng.uniform(0.001, 1, n))
    q = _t(rng.standard_normal((nvec, n)))
    plan = F.HalfPlaneFMM(x, y, 1.0 + 0.5j, p=20, leaf_size=20)
    one = torch.stack([plan(q[v]) for v in range(nvec)])  # a pass of one vector each
    alloc_hook("1+")
    with pytest.raises(F.FMMHPError) as e:  # the double layer's sorted normals: the hook tells their number
        plan.double_layer(q[0], q[0], q[0])
    assert e.value.status == 3
    if fail == "first":
        alloc_hook(str(int(re.search(r"array (\d+)", str(e.value)).group(1)) + 1))
    held = plan.info()["device_bytes"]
    got = plan(q)
    if fail == "1+":
        assert plan.info()["device_bytes"] == held
    grown = plan.info()["device_bytes"]
    for _ in range(3):
        assert torch.equal(plan(q), got)
    assert plan.info()["device_bytes"] == grown
    plan.close()
    assert torch.equal(got, one)

