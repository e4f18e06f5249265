"""The coarse operator and the coarse BiCGStab over their launch shapes.

The operator takes 8 columns of a block row at a time, for 8 RHS (or one alone) and,
where the rows leave waves over, for 16 or 32; its product is compared with the dense
matrix of the library's own stencil blocks, from the smallest to the largest coarse space
and around the group's size.  Each entry is a sum
of 9 ncv products in double precision: n eps of the sum of their sizes, n = 18 ncv.
The coarse solve's sums come from partials that the kernel before left: an RHS's bits
depend neither on its neighbours nor on a call before, and an RHS that is zero, or done
early, leaves the others alone.  Above 1024 coarse sites the partials are added in two
steps; there the solve is compared with the oracle's on the library's operator, at the
1e-9 that the small coarse spaces are held to.
"""
import numpy as np
import pytest

import laph_synth as ls
from gpu_common import dev, host, log_case, make_lattice, per_rhs_rel, require_gpu
from oracle import multigrid as omg
from test_gpu_mg import _dense_from_blocks

pytestmark = pytest.mark.gpu

DIMS, BLOCK = (4, 4, 4, 6), (2, 2, 2, 2)


def _lattice(nv, dims=DIMS):
    require_gpu()
    lat = make_lattice(dims, ls.gauge_field(dims, 71), masses=(0.1,))
    lat.mg_setup(dev(ls.random_spinor((nv,) + ls.spinor_shape(dims), 7100 + nv)), BLOCK, null_passes=0)
    return lat


@pytest.mark.parametrize("nv,ns", [(1, (1, 8, 65)), (4, (1, 31, 32, 33)), (5, (1, 15, 17)), (8, (2, 16)),
                                   (12, (8, 43)), (15, (16,)), (16, (1, 31, 32))])
def test_coarse_apply_groups(nv, ns):
    lat = _lattice(nv)
    C = host(lat.mg_coarse_matrix())
    D, size = _dense_from_blocks(C, DIMS, BLOCK), np.abs(_dense_from_blocks(np.abs(C), DIMS, BLOCK))
    for n in ns:
        log_case("coarse apply", nv=nv, n=n)
        c = ls.random_spinor((n, 3, 2, 2, 2, 2, nv), 7200 + n)
        got = host(lat.mg_coarse_apply(dev(c))).reshape(n, -1)
        flat = c.reshape(n, -1)
        bound = 36 * nv * 2.3e-16 * (np.abs(flat) @ size.T)
        assert (np.abs(got - flat @ D.T) <= bound).all()


@pytest.mark.parametrize("nv,n", [(1, 3), (4, 40), (8, 19), (12, 5), (16, 33)])
def test_coarse_solve_rhs_are_independent(nv, n):
    lat = _lattice(nv)
    c = ls.random_spinor((n, 3, 2, 2, 2, 2, nv), 7300 + n)
    c[1] = 0
    c[2] *= 1e-30
    log_case("coarse solve", nv=nv, n=n)
    got = host(lat.mg_component(3, dev(c)))
    assert np.isfinite(got).all() and (got[1] == 0).all()
    for r in sorted({0, 1, 2, n - 1}):
        log_case("coarse solve alone", r=r)
        assert np.array_equal(host(lat.mg_component(3, dev(c[r:r + 1])))[0], got[r])


class _Coarse:
    def __init__(self, lat, shape):
        self.lat, self.shape = lat, shape

    def __matmul__(self, x):
        return host(self.lat.mg_coarse_apply(dev(x.reshape((1,) + self.shape)))).ravel()


# coarse extents 8 x 8 x 4 x 4 (1024 sites, the last summed in one step) and 6^4
@pytest.mark.parametrize("dims", [(16, 16, 8, 8), (12, 12, 12, 12)])
def test_coarse_solve_many_sites(dims):
    nv, n = 2, 9
    lat = _lattice(nv, dims)
    shape = (dims[3] // 2, dims[2] // 2, dims[1] // 2, dims[0] // 2, 2, nv)
    c = ls.random_spinor((n,) + shape, 7400)
    D = _Coarse(lat, shape)
    log_case("coarse solve", dims=dims)
    got = host(lat.mg_component(3, dev(c)))
    pick = (0, 7, 8)
    ref = np.stack([omg.coarse_bicgstab(D, c[i].ravel(), 16, 0.1).reshape(shape) for i in pick])
    assert per_rhs_rel(got[list(pick)], ref).max() < 1e-9
