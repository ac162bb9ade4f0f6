"""GPU: moments past the largest number.  With |H| set below the spectrum the
Chebyshev moments of a plane wave of rescaled energy cosh(theta) are
cosh(n theta): infinite from order 710.4758 / theta on (cosh z > 2^1024).  The
correlation at time j sums the orders up to N(x_j) and no others, so it is
finite exactly where N(x_j) lies below that order (set half an order away from
a whole one: the sums that make the moments are rounded by parts in 2^40)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(csp):
    c = csp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("last", [400, 403, 406, 409, 412])
def test_times_before_an_infinite_moment_stay_finite(csp, ctx, last):
    print("[gpu] moments last finite order %d" % last, flush=True)
    theta = 710.4758 / (last + 0.5)
    g = csp.Lattice(ctx, "square", 64, 64, t=1.0, halfwidth_override=4.0 / math.cosh(theta))
    psi = torch.full((4096, 1), 1.0 / 64.0, dtype=torch.complex128, device="cuda:0")
    Nt = 136
    corr, _ = csp.csp_propagate(ctx, g, psi, csp.make_params(
        Nt, mode="fp64_conc", assembly=csp.CSP_ASSEMBLE_MOMENTS))
    finite = torch.isfinite(torch.view_as_real(corr)).all(dim=2).all(dim=1).cpu().numpy()
    orders = [csp.csp_chebyshev_coefficients(ctx, j * math.pi, 8)[1] for j in range(1, Nt + 1)]
    expect = np.array([True] + [n <= last for n in orders])
    assert expect.any() and not expect.all()
    assert np.array_equal(finite, expect)
    g.close()
