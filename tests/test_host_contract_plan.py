"""The rule that sends doublets by planes, against times of both ways measured on an MI355X (us, one
call): few planes leave the chip idle, a workgroup count just above a multiple of the 256 CUs
costs a whole round, a Hermitian plane alone saves little, small nev takes the time of a
16-block, and what a group saves depends on the momenta that stay."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# lx ly lz lt, nev, momenta of one (px, py), Hermitian, with the whole phase, by planes
MEASURED = [
    (48, 48, 4, 4, 64, 2, 1, 211, 1362), (32, 32, 4, 4, 64, 8, 1, 331, 622), (32, 32, 8, 8, 64, 1, 1, 192, 625),
    (32, 32, 8, 8, 64, 4, 0, 583, 631), (24, 24, 16, 18, 64, 1, 1, 427, 532), (24, 24, 16, 18, 64, 2, 0, 761, 583),
    (24, 24, 20, 26, 64, 1, 1, 690, 834), (30, 18, 14, 26, 64, 3, 1, 1249, 509), (16, 16, 8, 12, 64, 2, 1, 158, 181),
    (16, 16, 8, 12, 64, 8, 1, 469, 186), (16, 16, 16, 32, 64, 1, 1, 328, 262), (32, 32, 32, 64, 64, 1, 1, 3890, 3537),
    (32, 32, 32, 64, 64, 2, 0, 7715, 3895), (32, 32, 32, 64, 16, 2, 1, 2275, 1163), (12, 12, 12, 24, 64, 2, 0, 241, 175),
    (10, 22, 16, 24, 32, 4, 0, 436, 178), (8, 8, 8, 8, 64, 1, 0, 64, 73), (20, 24, 18, 40, 48, 4, 0, 2237, 607),
]


# the same for several groups: (momenta, Hermitian) of each, and all of them one way or the other
SEVERAL = [
    ((8, 8, 16, 32, 64), [(2, 1), (2, 0), (2, 0), (2, 0)], 549, 335),
    ((32, 32, 8, 8, 8), [(3, 1), (6, 0), (6, 0), (6, 0), (6, 0)], 1061, 1275),
    ((12, 12, 12, 24, 64), [(2, 1), (2, 0), (2, 0), (2, 0)], 729, 615),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_rule_takes_the_faster_way(tmp_path):
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", os.path.join(ROOT, "tests", "host", "contract_plan_check.cpp"),
                        "-o", exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    cases = [(m[:5], [m[5:7]], m[7], m[8]) for m in MEASURED] + SEVERAL
    lines = "".join("%d %d %d %d %d %d %s\n" % (d + (len(g), " ".join("%d %d" % x for x in g))) for d, g, _, _ in cases)
    r = subprocess.run([exe], input=lines, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    assert [int(v) for v in r.stdout.split()] == [len(g) if planes < whole else 0 for _, g, whole, planes in cases]
