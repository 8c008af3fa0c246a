"""The 256 x 256 byte contraction issues its matrix-core ops from blocks of
inline assembly that end before the last sums are written, so the compiler must
not put an instruction that reads or writes an accumulator between two blocks:
it does not know that one would have to wait.  (A wait inside the blocks, 11
states, cost 1.5% of a call on byte frames: 1539 -> 1563 us.)  This reads the
assembly that the compiler makes of the source: from the end of every run of
matrix ops, along every branch, nothing but matrix ops touches the run's
accumulators for 11 wait states, the most that ops of 8 passes need."""
import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WAIT = 11


def _regs(text):
    r = set()
    for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        r |= set(range(int(lo), int(hi) + 1))
    return r | {int(x) for x in re.findall(r"\bv(\d+)\b", text)}


def _violations(lines):
    """Instructions of a function's lines that touch an accumulator too early."""
    code, label = [], {}
    for ln in lines:
        ln = ln.split(";")[0].strip()
        if re.match(r"^[.\w$]+:$", ln):
            label[ln[:-1]] = len(code)
        elif ln and not ln.startswith("."):
            code.append(ln)
    is_mfma = [c.startswith("v_mfma") for c in code]
    bad, runs, i = [], 0, 0
    while i < len(code):
        if not is_mfma[i]:
            i += 1
            continue
        acc = set()
        while i < len(code) and is_mfma[i]:
            acc |= _regs(code[i].split(",")[0])
            i += 1
        runs += 1
        todo, seen = [(i, WAIT)], {}
        while todo:
            k, left = todo.pop()
            while left > 0 and k < len(code) and not is_mfma[k] and seen.get(k, 0) < left:
                seen[k] = left
                c = code[k]
                if _regs(c) & acc:
                    bad.append(c)
                op = c.split()[0]
                left -= int(c.split()[1], 0) + 1 if op == "s_nop" else 1
                if op.startswith("s_cbranch") or op == "s_branch":
                    todo.append((label[c.split()[1]], left))
                if op in ("s_branch", "s_endpgm"):
                    break
                k += 1
    return runs, bad


def test_finds_a_copy():
    mfma = "v_mfma_i32_16x16x64_i8 v[0:3], v[8:11], v[12:15], v[0:3]"
    assert _violations([mfma, "s_waitcnt lgkmcnt(0)", "s_nop 9", "v_mov_b32 v20, v1"]) == (1, [])
    assert _violations([mfma, "s_nop 9", "v_mov_b32 v20, v1"])[1] == ["v_mov_b32 v20, v1"]
    assert _violations([mfma, "s_cbranch_scc1 L", "s_nop 15", "s_endpgm", "L:",
                        "v_mov_b32 v2, v9"])[1] == ["v_mov_b32 v2, v9"]


def test_byte_contraction_waits(tmp_path):
    spec = importlib.util.spec_from_file_location(
        "_cpi_build", os.path.join(ROOT, "paper_2407_20692_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    try:
        hipcc = b.hipcc()
    except RuntimeError:
        pytest.skip("needs hipcc")
    out = str(tmp_path / "gemm.s")
    subprocess.run([hipcc] + b.FLAGS + ["-x", "hip", "--cuda-device-only", "-S",
                                        os.path.join(b.CSRC, "kernels_gemm.hip"), "-o", out],
                   check=True, capture_output=True, text=True, timeout=300)
    with open(out) as f:
        text = f.read()
    kernels = re.findall(r"^(_ZN\S*k_gemm_bytes_big\S*):[^\n]*\n(.*?)^\.Lfunc_end", text,
                         re.M | re.S)
    assert len(kernels) == 5   # one per mode
    for name, body in kernels:
        runs, bad = _violations(body.splitlines())
        assert runs == 3 and not bad, (name, runs, bad)
