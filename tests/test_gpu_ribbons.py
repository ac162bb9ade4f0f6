"""GPU: complex128 lattices open in y: launches of four steps (wide ribbons,
whose eight-step launches mostly compute margin rows, and lattices in segments
of four rows) or eight (few waves, larger lattices, or periodic in y), with the
same results.  The state
form's values do not depend on the steps of a launch; the sums of the moment
form are taken over other groups of rows, in FP64: 1e-12 of |psi|^2 = 1."""
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


# steps per launch of the moment form and of the states
@pytest.mark.parametrize("kind,Lx,Ly,py,msteps,ssteps", [
    ("honeycomb", 60000, 4, False, 4, 4), ("honeycomb", 60000, 1, False, 4, 4),
    ("square", 120001, 6, False, 4, 4), ("square", 120000, 2, False, 4, 4),
    ("square", 120000, 7, False, 4, 8), ("square", 120000, 4, True, 8, 8),
    ("honeycomb", 700, 4, False, 8, 8), ("square", 120000, 1, False, 8, 8),
    ("square", 560, 560, False, 4, 4), ("square", 560, 560, True, 8, 8),
    ("square", 700, 700, False, 4, 8), ("square", 300, 300, False, 8, 8),
    ("square", 1300, 1300, False, 8, 8)])
def test_ribbon_steps(csp, ctx, kind, Lx, Ly, py, msteps, ssteps):
    print("[gpu] ribbon %s %dx%d" % (kind, Lx, Ly), flush=True)
    g = csp.Lattice(ctx, kind, Lx, Ly, t=1.0, W=0.7, disorder_seed=2, periodic_y=py)
    R, Nt = 2, 12
    N = g.info.n_orb
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    ph = torch.rand((N, R), dtype=torch.float64, device="cuda:0", generator=gen) * (2 * np.pi)
    psi = torch.polar(torch.full_like(ph, N ** -0.5), ph)
    for assembly, b, steps in ((1, 0, msteps), (0, 7, ssteps)):
        params = csp.make_params(Nt, mode="fp64_conc", block_b=b, assembly=assembly)
        corr, rep = csp.csp_propagate(ctx, g, psi, params)
        assert rep.spmm_steps == steps, assembly
        other = csp.Context(0)
        T = csp.Tuning()
        T.spmm_vec, T.spmm_steps, T.spmm_seg_rows = 2, 12 - steps, 16
        T.contract_wg_per_cu, T.block_b = 4, b
        h = csp.Lattice(other, kind, Lx, Ly, t=1.0, W=0.7, disorder_seed=2, periodic_y=py)
        csp.csp_set_tuning(other, [h], [R], params, T)
        ref, rep = csp.csp_propagate(other, h, psi, params)
        assert rep.spmm_steps == 12 - steps
        assert (corr - ref).abs().max().item() < 1e-12
        h.close()
        other.close()
    E = [-0.5, 0.4]
    qe, rep = csp.csp_quasi_eigenstates(ctx, g, psi, csp.make_params(6, mode="fp64_conc"), E)
    assert rep.spmm_steps == ssteps
    # the sequential form: the ring and the contraction for one or two such rows
    ring = ssteps == 4 and Ly <= 2
    seq, rep = csp.csp_propagate(ctx, g, psi, csp.make_params(Nt, mode="fp64_seq"))
    assert (rep.contract_launches > 0) == ring
    assert (seq - corr).abs().max().item() < 1e-12
    g.close()
