"""The launch shapes that the tuner times (internal.hpp, compiled for the CPU): the plan's own default is the
first of them, whatever it is, and no two launch the same grid of the same kernel."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2507_21913_amd", "csrc")
HIPCC = "/opt/rocm/bin/hipcc"

DRIVER = r"""
#include <stdio.h>
#include "internal.hpp"
int main() {
    for (int cus : {256, 104})
        for (int nrec : {1, 40, 1000, 4096, 4097, 20000, 32767, 32768, 90000})
            for (int walk = 1; walk <= 4; ++walk)
                for (int groups = 1; groups <= 16; ++groups) {
                    printf("%d %d %d %d:", cus, nrec, walk, groups);
                    for (auto a : fmmhp::tune_shapes({walk, groups}, nrec, cus)) printf(" %d,%d", a.walk, a.groups);
                    printf("\n");
                }
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc is needed")
def test_default_first_and_no_duplicates(tmp_path):
    src, exe = tmp_path / "shapes.hip", tmp_path / "shapes"
    src.write_text(DRIVER)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", f"-I{CSRC}", str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    lines = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()
    assert len(lines) == 2 * 9 * 4 * 16
    for line in lines:
        head, tail = line.split(":")
        cus, nrec, walk, groups = map(int, head.split())
        shapes = [tuple(map(int, a.split(","))) for a in tail.split()]
        assert shapes[0] == (walk, groups)

        def launch(a):  # kernel and workgroups
            return (1, min((nrec + 3) // 4, a[1] * cus)) if a[0] <= 2 else (a[0], a[1] * cus)

        launches = [launch(a) for a in shapes]
        assert len(set(launches)) == len(launches), line
        for c in ((1, 2), (1, 4), (1, 8), (4, 4), (4, 8)):
            assert launch(c) in launches, line
    # a plan of 32,768 records below p = 30: its default is eight workgroups per CU
    assert "256 32768 1 8: 1,8 1,2 1,4 4,4 4,8" in lines
