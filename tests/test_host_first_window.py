"""Where a solve may take its first residual to live: the residual's support, followed hop by
hop on a line of timeslices, must lie in the window.  b_hat of a source on t0 reaches t0 +- 1;
with a nonzero x to start from, r = b_hat - M_hat x is nonzero wherever x or its
neighbours are, and a solve that took it for confined would drop sites."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _spread(slices, lt, hops):
    for _ in range(hops):
        slices = {(t + d) % lt for t in slices for d in (-1, 0, 1)}
    return slices


def test_first_residual_lies_in_its_window(tmp_path):
    if not (os.path.exists(HIPCC) or shutil.which("hipcc")):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "check")
    r = subprocess.run([HIPCC, "-std=c++17", "--offload-arch=gfx950", "-O1", "-x", "hip",
                        os.path.join(ROOT, "tests", "host", "first_window_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    cases = [(dims, t0, one, x) for dims in [(4, 4, 4, 12), (6, 4, 2, 10), (4, 4, 4, 4), (4, 4, 4, 2)]
             for t0 in range(dims[3]) for one in (0, 1) for x in (0, 1)]
    lines = "".join("%d %d %d %d %d %d %d\n" % (d + (t0, one, x)) for d, t0, one, x in cases)
    r = subprocess.run([exe], input=lines, capture_output=True, text=True, timeout=60)
    assert r.returncode == 0
    for (dims, t0, one, x), ln in zip(cases, r.stdout.splitlines()):
        lo, n = (int(v) for v in ln.split())
        lt, per = dims[3], dims[0] * dims[1] * dims[2] // 2
        every = set(range(lt))
        window = every if n == 0 else {((lo + d) % (lt * per)) // per for d in range(n)}
        b_hat = _spread({t0}, lt, 1) if one else every
        support = b_hat | (_spread(every, lt, 2) if x else set())
        assert support <= window
        if one and not x:
            assert window == b_hat   # and no wider than it has to be
