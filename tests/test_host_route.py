"""Builds the rule that takes stacks by direct gathers with g++ (address and
undefined-behaviour sanitizers), runs its host tests, and checks that the GPU
tests of the gathers reach them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_20692_amd", "csrc")


def test_gather_rule(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path / "route_test")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", CSRC,
                    os.path.join(CSRC, "refocus_route.cpp"),
                    os.path.join(ROOT, "tests", "host", "route_test.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "route tests passed" in r.stdout, r.stderr
    from tests.test_gpu_refocus_gather import CASES
    taken = []
    for g, al in CASES:
        args = [g.wa, g.ha, g.wb, g.hb, g.out_w, g.out_h, len(al), al[0], al[-1], 0]
        r = subprocess.run([exe] + [str(v) for v in args], capture_output=True, text=True,
                           timeout=60, check=True)
        taken.append(int(r.stdout))
    # all but the one with more views than the LDS holds, the small stacks just
    # beyond, and one plane too many
    assert taken == [1, 1, 1, 1, 1, 1, 0, 0, 0, 1, 1, 0, 1]
