"""The shapes that the multi-step grid kernels' tuners time, built by g++ and
checked over many grids and batches (tests/grid_shapes_main.cpp). CPU only."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1911_07065_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_shape_lists(tmp_path):
    exe = str(tmp_path / "grid_shapes")
    cmd = ["g++", "-std=c++17", "-O2", os.path.join(CSRC, "grid_shapes.cpp"),
           os.path.join(ROOT, "tests", "grid_shapes_main.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-2000:]
