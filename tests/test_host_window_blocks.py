"""The block range a windowed launch walks (and its reduction sums), against the per-block
test of the kernels, over every window of small lattices: whole and ragged last blocks,
windows that wrap, that cover the lattice, and none."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_window_blocks_names_the_blocks_that_overlap(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "window_blocks_check")
    src = os.path.join(ROOT, "tests", "host", "window_blocks_check.cpp")
    r = subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "-O1", "-x", "hip", src, "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    cases = [(64, 8), (60, 8), (61, 7), (30, 64), (57, 16), (96, 32)]
    r = subprocess.run([exe], input="".join("%d %d\n" % c for c in cases), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and [int(v) for v in r.stdout.split()] == [0] * len(cases)
