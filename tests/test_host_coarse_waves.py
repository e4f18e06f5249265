"""The coarse BiCGStab's kernels decide per workgroup: run on the CPU as fibers, with some
waves of a late workgroup before and the others after the workgroup that writes the RHS's
scalars, no wave leaves another at a barrier and no bit depends on the order.  Solves that
end in the p update, in the s update and before the first iteration."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.join(ROOT, "tests", "host")


def _kernels():
    """The solve's kernels and what they call, cut out of the multigrid's source."""
    with open(os.path.join(ROOT, "paper_2510_26313_amd", "csrc", "mg.hip")) as f:
        src = f.read()

    def cut(first, end, start=0):
        a = src.index(first, start)
        return src[a:src.index(end, a)]

    a = src.rindex("template", 0, src.index("void block_sum_bcast("))
    return "\n".join([cut("constexpr int kMB =", "\n"), src[a:src.index("\n}\n", a) + 3],
                      cut("struct CgState {", "constexpr int kCoarseRhs"),
                      cut("__device__ __forceinline__ void cg_sum(", "__global__ __launch_bounds__(kMB) void mg_mr_update")])


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_no_order_of_waves_matters(tmp_path):
    inc, exe = str(tmp_path / "kernels.inc"), str(tmp_path / "check")
    with open(inc, "w") as f:
        f.write(_kernels())
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-Wno-unknown-pragmas", '-DKERNELS="%s"' % inc,
                        os.path.join(HERE, "coarse_waves_check.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "0", r.stderr[-2000:]
