"""The FP32 launchers refuse the FP64-only row mode instead of launching
nothing and reporting success: a host program linked to the built library."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1004_1122_amd")


def test_fp32_launchers_refuse_fused_out(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "liblshom.so")):
        pytest.skip("liblshom.so not built")
    exe = tmp_path / "fused_out_check"
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(PKG, "csrc"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "fused_out_check.cpp"),
                    "-o", str(exe), "-L", PKG, "-llshom", f"-Wl,-rpath,{PKG}"], check=True, capture_output=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
