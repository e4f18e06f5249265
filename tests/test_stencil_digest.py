"""The digest that keys saved tuner choices and counter summaries covers the sources that
define the stencil's workgroup sizes."""
import os
import re

import bench
from paper_2510_26313_amd import build


def _defining(name):
    pat = re.compile(r"^constexpr int %s = " % name, re.M)
    return {f for f in os.listdir(build.CSRC) if f.endswith((".h", ".hip"))
            and pat.search(open(os.path.join(build.CSRC, f)).read())}


def test_workgroup_sizes_are_in_the_digest():
    for name in ("kBlock", "kLdsSites"):
        files = _defining(name)
        assert len(files) == 1
        assert files <= set(build.STENCIL_SOURCES) and files <= set(bench.STAGE_SOURCES)
