"""K slices of the triplets: enough workgroups where the lattice gives them, and never slices so
short that summing them (six reads an entry) outweighs the products they save: four chunks at
least, once there are four slices."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_slices_are_not_too_short(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(ROOT, "tests", "host", "triplet_split_check.cpp"),
                        "-o", exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    cases = [(base, n) for base in (1, 4, 32, 64, 200, 2048, 5000) for n in (1, 2, 3, 4, 7, 8, 15, 16, 27, 64, 216, 1728, 4096)]
    r = subprocess.run([exe], input="".join("%d %d\n" % c for c in cases), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    for (base, n), s in zip(cases, (int(v) for v in r.stdout.split())):
        assert 1 <= s <= min(n, 64)
        assert s <= 4 or n // s >= 4
        assert base * s >= 2048 or s in (64, min(n, 4), n // 4)
