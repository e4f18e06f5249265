"""The clover term built on the device (one wave per plane on 64 sites) against the
oracle, on lattices whose site count per parity leaves the last block full, nearly empty
and nearly full.  Products of six SU(3) factors summed over four leaves and two planes:
about 100 roundings of values of order one, so 1e-13 relative to the field."""
import numpy as np
import pytest

import laph_synth as ls
from gpu_common import dev, host, log_case, make_lattice, parity_mask, rel, require_gpu
from oracle import dirac

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (6, 4, 4, 10), (10, 6, 4, 4), (6, 6, 6, 6)])
def test_clover_term(dims):
    require_gpu()
    U = ls.gauge_field(dims, 71)
    psi = ls.random_spinor(ls.spinor_shape(dims, 2), 72)
    log_case("clover_build", dims=dims)
    lat = make_lattice(dims, U, masses=(0.1,), csw=1.3)
    A = dirac.clover_matrix(U, 0.1, 1.3)
    want = dirac.apply_site_matrix(A, psi)
    mask = parity_mask(dims)[None, ..., None, None]
    for parity in (0, 1):
        buf = lat.pack(dev(psi), "f64", parity)
        got = host(lat.unpack(lat.apply_clover(buf, 2, parity), 2, "f64", parity))
        assert rel(got * (mask == parity), want * (mask == parity)) < 1e-13
        inv = host(lat.unpack(lat.apply_clover(buf, 2, parity, inverse=True), 2, "f64", parity))
        back = dirac.apply_site_matrix(A, inv * (mask == parity))
        assert rel(back, psi * (mask == parity)) < 1e-12
