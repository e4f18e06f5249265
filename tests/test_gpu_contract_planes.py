"""Doublets whose momenta share their plane products, and triplets over the block table of
pairs, against the oracle: planes that are not whole chunks of 8 sites, vectors that do
not fill their 16-blocks, momenta of one (px, py) with both signs, (px, py) equal to its own
negative (a Hermitian plane), more momenta than one summing launch takes, and momenta that stay
on the full-phase path beside them.  Sums of n = 3 Lx Ly Lz products of normal values: the
rounding error is about sqrt(n) 1e-16 of the largest entry's n; the contraction tests'
1e-12 of the largest entry covers it."""
import numpy as np
import pytest

import laph_synth as ls
from gpu_common import dev, host, log_case, require_gpu
from oracle import laph as olaph

pytestmark = pytest.mark.gpu


def _close(got, ref):
    assert np.abs(got - ref).max() <= 1e-12 * np.abs(ref).max()


# (nx, ny) = (0, 0) and (L/2, 0) are their own negatives; (1, 2) comes with both signs
PLANE_MOMS = [(0, 0, 0), (0, 0, 1), (0, 0, -3), (1, 2, 0), (-1, -2, 0), (1, 2, 2), (-1, -2, 5), (2, 0, 1)]


@pytest.mark.parametrize("dims,nev", [((18, 14, 20, 12), 64), ((16, 16, 12, 16), 50), ((10, 22, 16, 24), 33)])
def test_doublets_by_planes(dims, nev):
    require_gpu()
    import paper_2510_26313_amd as laph
    lx, ly, lz, lt = dims
    V = ls.random_spinor((lt, nev, lz, ly, lx, 3), 900 + nev)
    moms = PLANE_MOMS + [(lx // 2, 0, 1), (-lx // 2, ly, -2)] + [(0, 0, k) for k in range(4, 12)]
    # what decides for a group: the products saved take longer than about 40 us at 50 TFLOP/s
    assert 8 * 3 * lx * ly * lz * lt * nev ** 2 / 50e12 > 40e-6
    log_case("doublets_by_planes", dims=dims, nev=nev, moms=len(moms))
    lat = laph.Lattice(dims)
    got = host(lat.meson_doublets(dev(V), moms))
    ref = np.concatenate([olaph.meson_doublets(V[t:t + 1], moms) for t in range(lt)], axis=1)
    _close(got, ref)


@pytest.mark.parametrize("nev", [15, 16, 17, 33, 48, 50])
def test_triplet_pairs(nev):
    require_gpu()
    import paper_2510_26313_amd as laph
    dims = (4, 4, 4, 4)
    V = ls.random_spinor((4, nev, 4, 4, 4, 3), 950 + nev)
    moms = [(0, 0, 0), (1, -1, 2)]
    log_case("triplet_pairs", nev=nev)
    got = host(laph.Lattice(dims).baryon_triplets(dev(V), moms))
    _close(got, olaph.baryon_triplets(V, moms))
    assert np.array_equal(got, -np.swapaxes(got, 2, 3)) and np.array_equal(got, -np.swapaxes(got, 3, 4))
