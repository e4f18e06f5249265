"""Doublets on the ways the launch rule picks, against the oracle: fewer vectors than a 16-block and
planes, planes on a lattice of few timeslices, and the whole phase where planes would leave the
chip idle.  Bound as in the other contraction tests: 1e-12 of the largest entry."""
import numpy as np
import pytest

import laph_synth as ls
from gpu_common import dev, host, log_case, require_gpu
from oracle import laph as olaph

pytestmark = pytest.mark.gpu

MOMS = [(0, 0, 0), (0, 0, 1), (0, 0, -3), (1, 2, 0), (-1, -2, 1), (1, 2, 2), (2, 0, 1)]


@pytest.mark.parametrize("dims,nev", [((20, 18, 16, 32), 3), ((20, 18, 16, 32), 17), ((16, 16, 16, 4), 64),
                                      ((32, 32, 4, 4), 64), ((10, 12, 14, 18), 1)])
def test_doublet_routes(dims, nev):
    require_gpu()
    import paper_2510_26313_amd as laph
    lx, ly, lz, lt = dims
    V = ls.random_spinor((lt, nev, lz, ly, lx, 3), 960 + nev)
    log_case("doublet_routes", dims=dims, nev=nev)
    got = host(laph.Lattice(dims).meson_doublets(dev(V), MOMS))
    ref = np.concatenate([olaph.meson_doublets(V[t:t + 1], MOMS) for t in range(lt)], axis=1)
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()
