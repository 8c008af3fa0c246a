"""Builds the HIP-free plan of the register-window refocus with g++ (address
and undefined-behaviour sanitizers), runs its host tests, and checks that the GPU
tests of that pass reach it: the plan takes their cases (or not, for those of
wider windows), with each number of views staged among them, and they are above
the size that is gathered directly."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_20692_amd", "csrc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("window") / "window_test")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
           "-fno-sanitize-recover=all", "-I", CSRC, os.path.join(CSRC, "refocus_window_plan.cpp"),
           os.path.join(ROOT, "tests", "host", "window_test.cpp"), "-o", exe]
    subprocess.run(cmd, check=True, capture_output=True, text=True)
    return exe


def test_window_plan_with_sanitizers(exe):
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr
    assert "window tests passed" in r.stdout


def _split(exe, g, al):
    assert len(al) * g.out_w * g.out_h * g.wb * g.hb > 1 << 24, g
    assert g.wa >= 64, g
    args = [g.wa, g.ha, g.wb, g.hb, g.out_w, g.out_h, g.mag_x, g.mag_y, g.ca_x, g.ca_y, g.cb_x,
            g.cb_y] + list(al)
    r = subprocess.run([exe] + [repr(float(v)) for v in args], capture_output=True, text=True,
                       timeout=60, check=True)
    return r.stdout.split()


def test_gpu_cases_take_the_window_pass(exe):
    from tests.test_gpu_refocus_window_edges import CASES, WIDE
    from tests.test_gpu_refocus_window_far import CASES as FAR
    stages, shapes = set(), set()
    for g, al in CASES + FAR:
        s = [int(v) for v in _split(exe, g, al)]
        assert len(s) == 4, (g, s)
        shapes.add(tuple(s[:3]))
        stages.add(min(3, 9 // s[3]))
    assert stages == {1, 2, 3} and len(shapes) == 3
    for g, al in FAR:
        assert _split(exe, g, al)[3] == "9", g
    for g, al in WIDE:
        assert _split(exe, g, al) == ["none"], g
