"""The shapes of test_gpu_cnn_variants reach the kernels they are named for
(the launchers' own choice, asked on the host), and together they reach every
one the launchers can choose."""

import os
import shutil
import subprocess

import pytest

from paper_1004_1122_amd import cnn

variants = pytest.importorskip("test_gpu_cnn_variants")

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1004_1122_amd")
CONV3, DOWN3, POINT, DOWN3_T = 0, 1, 2, 3


def _query(case):
    op, index, c0, n, B = case
    name, hi, ho, cin, cout = cnn.layer_geometry(index, n, c0)
    cout8 = (cout + 7) // 8 * 8
    taps = 1 if name == "head" else 9
    if op == "wgrad":
        return f"wgrad {B} {ho} {cin} {cout8} {taps}"
    if op == "forward":
        mode = POINT if taps == 1 else (DOWN3 if name.startswith("down") else CONV3)
        return f"conv {mode} {3 if name.startswith('up') else 1} {B} {ho} {cin} {cout} {cout8}"
    mode = POINT if taps == 1 else (DOWN3_T if name.startswith("down") else CONV3)
    return f"conv {mode} 1 {B} {ho} {cout8} {cin} {cin}"


def test_cases_reach_their_kernels(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "liblshom.so")):
        pytest.skip("liblshom.so not built")
    exe = tmp_path / "cnn_variants"
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(PKG, "csrc"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "cnn_variants.cpp"),
                    "-o", str(exe), "-L", PKG, "-llshom", f"-Wl,-rpath,{PKG}"], check=True, capture_output=True)
    text = "\n".join(_query(c) for c, _ in variants.CASES) + "\n"
    out = subprocess.run([str(exe)], input=text, check=True, capture_output=True, text=True, timeout=60).stdout
    seen = set()
    for (case, want), line in zip(variants.CASES, out.strip().split("\n"), strict=True):
        v = [int(s) for s in line.split()]
        got = ("wgrad", *v) if case[0] == "wgrad" else (("patch", v[0], v[1]) if v[0] else ("wave", v[2], v[3]))
        assert got == want, (case, got)
        seen.add(got)
    assert seen == {("patch", 8, 1), ("patch", 8, 2), ("patch", 4, 2), ("wave", 4, 2), ("wave", 2, 2), ("wave", 4, 1),
                    ("wave", 2, 1), ("wave", 1, 1), ("wgrad", 64, 0), ("wgrad", 64, 1), ("wgrad", 32, 0),
                    ("wgrad", 32, 1)}
