"""Growth of a plan's workspaces within a recording of the caller's, compiled for the CPU against a stream that
records and a hipMalloc that refuses: calls take what is there, a first complex call is refused, and neither
narrows the plan's later calls."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_21913_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

SOURCE = r"""
#include <assert.h>
#include <stdio.h>
#include "workspace.hpp"
using namespace fmmhp;

static bool rec = false;
static int calls = 0;
static char *at = (char *)0x10000000000;
extern "C" hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) {
    *s = rec ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
extern "C" hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
extern "C" hipError_t hipMalloc(void **p, size_t n) {
    ++calls;
    if (rec) return hipErrorStreamCaptureUnsupported;
    *p = at;
    at += (n + 4095) / 4096 * 4096;
    return hipSuccess;
}
extern "C" hipError_t hipFree(void *) { return hipSuccess; }
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
extern "C" const char *hipGetErrorString(hipError_t) { return ""; }
namespace fmmhp { void set_error(const char *, ...) {} }

int main() {
    for (int nvec = 1; nvec <= 17; ++nvec) {
        Arena A;
        Tree T;
        Sched S;
        T.n = 200003;
        T.nbox = 20001;
        S.PB = 20;
        S.n_rch = 99;
        hipStream_t s = nullptr;
        rec = false;
        assert(ensure_vec_ws(A, T, S, 1) == FMMHP_OK);
        A.left = 0;
        rec = true;
        const int c = calls;
        assert(grow_eval_ws(A, T, S, nvec, s) == FMMHP_OK && S.ws.cap == 1 && calls == c);
        assert(grow_split(A, T, S, nvec, s) == FMMHP_ENOMEM && S.ccap == 0 && !S.cq && !S.cphi);
        rec = false;
        assert(grow_eval_ws(A, T, S, nvec, s) == FMMHP_OK && S.ws.cap == pass_width(nvec));
        assert(grow_split(A, T, S, nvec, s) == FMMHP_OK && S.ccap == std::min(nvec, 4));
        rec = true;
        const int d = calls;
        assert(grow_eval_ws(A, T, S, 17, s) == FMMHP_OK && S.ws.cap == pass_width(nvec) && calls == d);
        assert(grow_split(A, T, S, 17, s) == FMMHP_OK && S.ccap == std::min(nvec, 4) && calls == d);
    }
    printf("RECORDING_OK\n");
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc is needed")
def test_recording_allocates_nothing(tmp_path):
    src, exe = tmp_path / "rec.hip", tmp_path / "rec"
    src.write_text(SOURCE)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "RECORDING_OK" in r.stdout, r.stdout + r.stderr
