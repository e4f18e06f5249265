"""A reliable update ends with one finalize or, from 2^22 site-RHS on, with two (RHS that are done
are not lowered then): the same RHS solved in a batch of either kind have the same bits."""
import pytest
import torch

import laph_synth as ls
from gpu_common import dev, log_case, make_lattice, require_gpu

pytestmark = pytest.mark.gpu

DIMS, N, FEW = (16, 16, 16, 32), 70, 6   # 70 x 65536 sites per parity are above 2^22, 6 below


@pytest.mark.parametrize("stencil", [1, 2])
@pytest.mark.parametrize("prec", ["f16n", "f32", "f64"])
def test_batches_of_either_kind_agree(prec, stencil):
    require_gpu()
    import paper_2510_26313_amd as laph
    lat = make_lattice(DIMS, ls.gauge_field(DIMS, 91), masses=(0.05,))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(92)
    B = torch.complex(*(torch.randn(lat.spinor_shape(N), dtype=torch.float64, device="cuda", generator=gen) for _ in range(2)))
    p = dict(inner_prec=prec, stencil=stencil, rhs_tile=4, traversal=2, stencil64=2, rhs_tile64=4)
    log_case("update_finalize", **p)
    X, stats = lat.solve_raw(B, 0, params=laph.default_params(**p))
    few, want = lat.solve_raw(B[N - FEW:].clone(), 0, params=laph.default_params(**p))
    assert stats[N - FEW:] == want
    assert torch.equal(X[N - FEW:], few)
    assert max(s["true_res"] for s in stats) <= 1e-10
