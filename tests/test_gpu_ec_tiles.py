"""GPU: column tiles of the complex128 conductivity moments against the oracle.

The moment kernel packs the real and imaginary columns of a tile's energies
into 16-column matrix tiles, one to seven of them, and splits more than 56
energies over several tiles.  Energy counts at the edges of every tile count,
on a lattice whose slices end inside a staged step of 16 orbitals and whose
last chunk of orders ends inside a wave's 32.  Tolerance as for every
complex128 conductivity test: 1e-10 of the largest correlation (sums of at
most 1073 products of order 1 / 1073, an error of a few 1e-15 of it)."""
import numpy as np
import pytest

import oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def setup():
    import paper_2510_17432_amd as csp
    ctx = csp.Context(0)
    spec = dict(t=1.0, W=0.9, disorder_seed=12)
    g = csp.Lattice(ctx, "square", 37, 29, **spec)       # 1073 sites: slices 512 + 512 + 49
    c = o.Lattice("square", 37, 29, **spec)
    yield csp, ctx, g, c
    g.close()
    ctx.close()


@pytest.mark.parametrize("n_E", [1, 7, 8, 9, 16, 24, 25, 40, 41, 48, 49, 56, 57, 100, 113, 128])
def test_energy_tiles(setup, n_E):
    csp, ctx, g, c = setup
    print("[gpu] EC tiles n_E %d" % n_E, flush=True)
    R, Nt = 2, 43                                        # 170 orders: chunks of 128 and 42
    rng = np.random.default_rng(n_E)
    psi = o.random_phase_states_fast(c.N, R, 5)
    # any states serve as bras; |<psi|Psi>| is kept away from zero
    qe = (rng.normal(size=(n_E, c.N, R)) + 1j * rng.normal(size=(n_E, c.N, R))) / np.sqrt(c.N)
    qe += 2.0 * psi[None]
    ref, _ = o.ec_correlation(c, psi, qe, Nt, 0, Hn=g.halfwidth)
    p, q = (torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0") for x in (psi, qe))
    corr, rep = csp.csp_ec_correlation(ctx, g, 0, p, q, csp.make_params(Nt, mode="fp64_conc"))
    torch.cuda.synchronize()
    assert rep.contract_launches == 2
    assert np.max(np.abs(corr.cpu().numpy() - ref)) < 1e-10 * np.max(np.abs(ref))
