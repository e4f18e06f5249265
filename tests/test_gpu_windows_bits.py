"""A perambulator's solves run their first iterations on the source's light cone and read r^ on
its slab; what is skipped is zero, and a windowed sum adds its partials in the places they have
in the whole one.  So no bit may differ from the general solve of the same sources, which
knows no source timeslice: equal iteration counts, updates, restarts and residuals for each
RHS, and equal perambulators.  With bursts of iterations shorter than the windowed phase;
with restarts inside that phase, which give r^ the whole lattice; and with a second pass, whose
residual is not confined."""
import numpy as np
import pytest
import torch

import laph_synth as ls
from gpu_common import dev, log_case, make_lattice, require_gpu

pytestmark = pytest.mark.gpu

NEV = 16   # 64 RHS: more than 2^20 site-RHS per batch on these lattices
RAGGED, WIDE = (10, 6, 14, 44), (16, 8, 8, 64)


def _setup(dims, m0, scale=1.0):
    require_gpu()
    assert int(np.prod(dims)) // 2 * 4 * NEV >= 1 << 20
    lat = make_lattice(dims, ls.gauge_field(dims, 81), masses=(m0,))
    return lat, dev(scale * ls.orthonormal_laph_vectors(dims, NEV, 82))


def _same(lat, V, t0, tol, **p):
    """The general solve's statistics, after comparing it with the perambulator bit for bit."""
    import paper_2510_26313_amd as laph
    p = dict(rhs_tile=4, traversal=2, **p)
    log_case("light_cone_bits", dims=lat.dims, t0=t0, tol=tol, **p)
    X, want = lat.solve_raw(lat.make_sources(V, t0), 0, tol, laph.default_params(**p))
    ref = lat.project_raw(X, V)
    tau, stats = lat.perambulator_raw(V, t0, 0, tol, laph.default_params(**p))
    assert stats == want
    assert torch.equal(tau, ref) and float(tau.abs().max()) > 0
    return want


@pytest.mark.parametrize("prec", ["f16n", "f32", "f64"])
@pytest.mark.parametrize("dims,t0,stencil", [(RAGGED, 43, 2), (RAGGED, 1, 1), (WIDE, 20, 2)])
def test_same_bits_as_the_general_solve(dims, t0, stencil, prec):
    lat, V = _setup(dims, 0.05)
    # the windowed phase: 5 iterations at 44 timeslices, 8 at 64
    for burst in (dict(), dict(graph_iters=2), dict(graph_iters=3, use_graph=0)):
        _same(lat, V, t0, 1e-10, inner_prec=prec, stencil=stencil, **burst)


# |r^|^2 is near 1e-160, so that |<r^, r>|^2 is no longer a double from the second iteration on: each of
# those is a breakdown and restarts from its residual (a CPU model of the solve gives 3 to 8 of the
# 10 restarts allowed to 5e-3)
@pytest.mark.parametrize("stencil", [1, 2])
def test_restarts_on_the_light_cone(stencil):
    lat, V = _setup(RAGGED, 0.05, 1e-79)
    stats = _same(lat, V, 7, 5e-3, inner_prec="f64", stencil=stencil)
    assert min(s["restarts"] for s in stats) >= 1


# At m0 = 20 the clover term is about 24, and an iteration gains 4 digits.  The solve stops at
# 0.2 tol on the even-odd residual, 1/24 of the whole one: with |r| / |b| = 2.3e-6 and 3.2e-10 after one
# and two iterations (a CPU model of the solve), these tolerances let the first pass end there and
# the whole residual miss.  maxiter ends the first pass at the latest then: one more
# iteration is the second pass's.
@pytest.mark.parametrize("stencil", [1, 2])
@pytest.mark.parametrize("prec,tol,first", [("f32", 2.4e-5, 1), ("f64", 3.5e-9, 2)])
def test_second_pass(prec, tol, first, stencil):
    lat, V = _setup(RAGGED, 20.0)
    stats = _same(lat, V, 40, tol, inner_prec=prec, stencil=stencil, maxiter=first)
    assert all(s["iters"] == first + 1 for s in stats)
