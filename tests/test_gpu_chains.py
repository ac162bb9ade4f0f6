"""GPU: single open rows (chains, and square lattices of one open row), whose
recursion launch runs without a row loop, against the FP64 oracle: lengths
below a strip, at its owned width and one site past it, odd ones (seams that
no wide access can take) and even ones, periodic and open ends, with and
without on-site energies, every steps-per-launch shape and every form.
Tolerances as for every launch shape: complex128 1e-10, complex64 2e-5 on
correlations, and five times those on the final states' largest element times
sqrt(N) (values of order 1 / sqrt(N))."""
import numpy as np
import pytest

import oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = {"fp32_conc": [(2, 1), (2, 4), (2, 8), (4, 2), (4, 8)],
          "fp64_conc": [(2, 1), (2, 2), (2, 4), (2, 8)]}
LENGTHS = [3, 50, 112, 113, 301, 482, 1000]


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(csp):
    c = csp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("W", [0.0, 0.9])
@pytest.mark.parametrize("periodic", [True, False])
@pytest.mark.parametrize("Lx", LENGTHS)
def test_chain_forms_match_oracle(csp, ctx, Lx, periodic, W):
    print("[gpu] chain %d periodic=%d W=%.1f" % (Lx, periodic, W), flush=True)
    R, Nt, b = 3, 22, 9
    kw = dict(t=1.0, W=W, disorder_seed=12, periodic_x=periodic)
    c = o.Lattice("chain", Lx, 1, **kw)
    psi = o.random_phase_states_fast(c.N, R, 31)
    lats = [csp.Lattice(ctx, "chain", Lx, **kw)]
    if Lx > 100:
        lats.append(csp.Lattice(ctx, "square", Lx, 1, periodic_y=False, **kw))
    for g in lats:
        ref, _, fin_ref = o.propagate(c, psi, Nt, b=0, return_final=True, Hn=g.halfwidth)
        for mode, shapes in SHAPES.items():
            fp64 = mode == "fp64_conc"
            p = torch.from_numpy(psi).to("cuda:0").to(torch.complex128 if fp64 else torch.complex64)
            tol = 1e-10 if fp64 else 2e-5
            for v, k in shapes:
                for assembly, blk in ((1, 0), (1, b), (0, b)):
                    if (v, k, assembly) == (4, 8, 1):
                        continue                     # no such moment kernel
                    params = csp.make_params(Nt, mode=mode, block_b=blk, assembly=assembly)
                    T = csp.Tuning()
                    T.spmm_vec, T.spmm_steps, T.spmm_seg_rows = v, k, 4
                    T.contract_wg_per_cu, T.block_b = 4, b
                    csp.csp_set_tuning(ctx, [g], [R], params, T)
                    fin = torch.zeros_like(p) if blk else None
                    corr, _ = csp.csp_propagate(ctx, g, p, params, final=fin)
                    torch.cuda.synchronize()
                    what = (g.info.rows, mode, v, k, assembly, blk)
                    assert np.max(np.abs(corr.cpu().numpy() - ref)) < tol, what
                    if blk:
                        d = np.max(np.abs(fin.cpu().numpy() - fin_ref)) * np.sqrt(c.N)
                        assert d < 5 * tol, what
        fin = torch.zeros_like(p)
        corr, rep = csp.csp_propagate(ctx, g, p, csp.make_params(Nt, mode="fp64_seq"), final=fin)
        torch.cuda.synchronize()
        assert rep.contract_launches == 0
        assert np.max(np.abs(corr.cpu().numpy() - ref)) < 1e-10
        assert np.max(np.abs(fin.cpu().numpy() - fin_ref)) < 1e-10
        g.close()
