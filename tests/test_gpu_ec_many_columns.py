"""GPU: conductivity of more columns than a grid's y or z dimension holds
(65536 groups of four): the columns are independent, so the call has to give
what calls of fewer columns give."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_many_states_and_energies():
    import paper_2510_17432_amd as csp
    ctx = csp.Context(0)
    g = csp.Lattice(ctx, "square", 8, 8, t=1.0, W=0.3, disorder_seed=2)
    R, nE, N, Nt = 2080, 128, 64, 3
    print("[gpu] ec %d columns" % (R * nE), flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(4)
    psi = torch.randn((N, R), dtype=torch.complex64, device="cuda:0", generator=gen)
    qe = torch.randn((nE, N, R), dtype=torch.complex64, device="cuda:0", generator=gen)
    p = csp.make_params(Nt, mode="fp32_conc")
    corr, _ = csp.csp_ec_correlation(ctx, g, 0, psi, qe, p)
    for lo, hi in ((0, 1056), (1056, 2080)):      # whole groups of 32 columns
        part, _ = csp.csp_ec_correlation(ctx, g, 0, psi[:, lo:hi].contiguous(),
                                         qe[:, :, lo:hi].contiguous(), p)
        assert torch.equal(part, corr[:, :, lo:hi])
    g.close()
    ctx.close()
