"""The default row-pass shape of small 3-D grids: one component per block, and
a block of a batch's launch holds at least 256 points (or as many rows as it
may, or the grid has), not the few rows that would give one small image many
blocks."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1004_1122_amd")
GRIDS = [(3, 3, 3), (5, 5, 5), (9, 8, 7), (12, 12, 12), (16, 16, 16), (20, 20, 20), (24, 24, 24), (30, 30, 30),
         (45, 45, 45), (60, 60, 60), (20, 30, 40), (40, 30, 20), (64, 32, 16), (4, 4, 200), (105, 77, 9), (11, 13, 17),
         (100, 100, 100), (105, 135, 77)]


def test_blocks_of_small_grids(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not os.path.exists(os.path.join(PKG, "liblshom.so")):
        pytest.skip("liblshom.so not built")
    exe = tmp_path / "row_shape"
    subprocess.run([hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-I", os.path.join(PKG, "csrc"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "native", "row_shape.cpp"),
                    "-o", str(exe), "-L", PKG, "-llshom", f"-Wl,-rpath,{PKG}"], check=True, capture_output=True)
    asked = [(g, elem) for g in GRIDS for elem in (16, 8)]
    out = subprocess.run([str(exe)], input="\n".join("%d %d %d %d" % (*g, e) for g, e in asked) + "\n", check=True,
                         capture_output=True, text=True, timeout=60).stdout
    for (grid, elem), line in zip(asked, out.strip().split("\n"), strict=True):
        rows, split, points, fits = map(int, line.split())
        assert split == 1 and fits == 1, (grid, elem)
        assert rows <= 64 and rows <= grid[0] * grid[1] + 1, (grid, elem, rows)
        assert points >= 256 or rows >= min(64, grid[0] * grid[1]), (grid, elem, rows, points)
