"""The block size that a pass launch takes when its schedule leaves it open:
four waves while a CU holds the launch's share of such blocks, three of the
FP64 kernels with a radix of 11, 13 or 17 and four of the others; two waves
where a block has no more points than two waves have lanes; four where two
cannot hold the butterflies or leave one idle."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1004_1122_amd")

# (n, points, LDS bytes, blocks, bytes): threads
CASES = [
    ((119, 238, 8000, 768, 16), 256),
    ((119, 238, 8000, 769, 16), 128),   # sixteen problems of 119^2: 960 blocks
    ((255, 510, 16000, 1024, 16), 128),
    ((143, 286, 9000, 864, 16), 128),
    ((119, 238, 4000, 1024, 8), 256),   # FP32
    ((119, 238, 4000, 1025, 8), 128),
    ((150, 300, 10000, 1024, 16), 256),
    ((150, 300, 10000, 1025, 16), 128),
    ((81, 81, 3000, 100, 16), 128),
    ((500, 1000, 24000, 5000, 16), 256),
    ((500, 1000, 12000, 5000, 8), 128),
    ((255, 2000, 40000, 5000, 16), 256),
]


def test_block_threads(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "liblshom.so")):
        pytest.skip("liblshom.so not built")
    exe = tmp_path / "block_threads"
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(PKG, "csrc"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "block_threads.cpp"),
                    "-o", str(exe), "-L", PKG, "-llshom", f"-Wl,-rpath,{PKG}"], check=True, capture_output=True)
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d %d %d" % c for c, _ in CASES) + "\n", check=True,
                         capture_output=True, text=True, timeout=60).stdout.split()
    assert [int(t) for t in out] == [t for _, t in CASES]
