"""GPU: the recursion kernel's two forms of a strip against the FP64 oracle.

A strip runs with whole lanes (wide accesses at one lane offset, no tests in
the steady rows) when every lane's values follow each other in memory and
every row is inside the lattice, and position by position otherwise.  These
lattices put both forms, and the change between them, at their edges: seams
of even and odd periodic rows, rows that are a multiple of two values but
not of four, open edges in x and y, segments long enough to have steady rows
and shorter than the margins, fewer rows than margin rows, a diagonal with
and without on-site energies.  Tolerances as for every launch shape:
complex128 1e-10, complex64 2e-5 on correlations, and five times those on
the final states' largest element times sqrt(N) (values of order 1 / sqrt(N))."""
import numpy as np
import pytest

import oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LATS = [
    dict(kind="square", Lx=246, Ly=70, t=1.0, W=0.8, disorder_seed=4),
    dict(kind="square", Lx=241, Ly=53, t=1.0, W=0.0),
    dict(kind="square", Lx=130, Ly=3, t=-1.0, W=0.6, disorder_seed=5),
    dict(kind="square", Lx=140, Ly=64, t=1.0, W=0.0, periodic_y=False, center=0.3),
    dict(kind="square", Lx=240, Ly=90, t=1.0, W=0.4, disorder_seed=8, periodic_x=False),
    dict(kind="honeycomb", Lx=65, Ly=66, t=-2.7, W=0.0),
    dict(kind="honeycomb", Lx=120, Ly=47, t=-2.7, W=1.0, disorder_seed=7),
    dict(kind="honeycomb", Lx=61, Ly=96, t=-2.7, W=0.5, disorder_seed=9, periodic_y=False),
]
SHAPES = {"fp32_conc": [(2, 1), (2, 2), (2, 4), (2, 8), (4, 4)],
          "fp64_conc": [(2, 1), (2, 2), (2, 4)]}


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(csp):
    c = csp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("spec", LATS)
def test_strip_forms_match_oracle(csp, ctx, spec):
    print("[gpu] strips %s %dx%d" % (spec["kind"], spec["Lx"], spec["Ly"]), flush=True)
    g = csp.Lattice(ctx, **spec)
    rest = {k: v for k, v in spec.items() if k not in ("kind", "Lx", "Ly", "center")}
    c = o.Lattice(spec["kind"], spec["Lx"], spec["Ly"], **rest)
    R, Nt, b = 2, 24, 9
    psi = o.random_phase_states_fast(c.N, R, 23)
    ref, _, fin_ref = o.propagate(c, psi, Nt, b=0, return_final=True, Hn=g.halfwidth,
                                  H0=spec.get("center", 0.0))
    for mode, shapes in SHAPES.items():
        fp64 = mode == "fp64_conc"
        p = torch.from_numpy(psi).to("cuda:0").to(torch.complex128 if fp64 else torch.complex64)
        tol = 1e-10 if fp64 else 2e-5
        for v, k in shapes:
            for seg in (8, 40):
                # one block by moments; time blocks of both assemblies with a final state
                for assembly, blk in ((1, 0), (1, b), (0, b)):
                    params = csp.make_params(Nt, mode=mode, block_b=blk, assembly=assembly)
                    T = csp.Tuning()
                    T.spmm_vec, T.spmm_steps, T.spmm_seg_rows = v, k, seg
                    T.contract_wg_per_cu, T.block_b = 4, b
                    csp.csp_set_tuning(ctx, [g], [R], params, T)
                    fin = torch.zeros_like(p) if blk else None
                    corr, _ = csp.csp_propagate(ctx, g, p, params, final=fin)
                    torch.cuda.synchronize()
                    what = (mode, v, k, seg, assembly, blk)
                    assert np.max(np.abs(corr.cpu().numpy() - ref)) < tol, what
                    if blk:
                        d = np.max(np.abs(fin.cpu().numpy() - fin_ref)) * np.sqrt(c.N)
                        assert d < 5 * tol, what
    g.close()


@pytest.mark.parametrize("tau", [np.pi, 0.01, 0.4, 7.0])
@pytest.mark.parametrize("spec", LATS)
def test_sequential_and_self_product_forms(csp, ctx, spec, tau):
    """The sequential form (carried state and <psi0|psi> in the recursion's
    epilogue; from 3 to 29 orders a step, so one launch, whole launches and
    remainders) and the complex128 self products at 8 steps per launch.  Both
    sum what the oracle sums in another order: 1e-10 as for complex128."""
    print("[gpu] seq %s %dx%d tau %.2f" % (spec["kind"], spec["Lx"], spec["Ly"], tau), flush=True)
    g = csp.Lattice(ctx, **spec)
    rest = {k: v for k, v in spec.items() if k not in ("kind", "Lx", "Ly", "center")}
    c = o.Lattice(spec["kind"], spec["Lx"], spec["Ly"], **rest)
    R, Nt = 3, 19                       # two batches of step records, groups of 2 and 1 columns
    psi = o.random_phase_states_fast(c.N, R, 29)
    kw = dict(Hn=g.halfwidth, H0=spec.get("center", 0.0), tau=tau)
    ref, _, fin_ref = o.propagate(c, psi, Nt, b=0, return_final=True, **kw)
    p = torch.from_numpy(psi).to("cuda:0")
    for norm in (False, True):
        fin = torch.zeros_like(p)
        corr, rep = csp.csp_propagate(ctx, g, p, csp.make_params(
            Nt, mode="fp64_seq", tau_tilde=tau, check_norm=norm), final=fin)
        torch.cuda.synchronize()
        assert rep.contract_launches == 0 and rep.n_blocks == Nt
        assert np.max(np.abs(corr.cpu().numpy() - ref)) < 1e-10
        assert np.max(np.abs(fin.cpu().numpy() - fin_ref)) < 1e-10
    for seg in (8, 40):
        params = csp.make_params(Nt, mode="fp64_conc", tau_tilde=tau,
                                 assembly=csp.CSP_ASSEMBLE_MOMENTS)
        T = csp.Tuning()
        T.spmm_vec, T.spmm_steps, T.spmm_seg_rows, T.contract_wg_per_cu = 2, 8, seg, 4
        csp.csp_set_tuning(ctx, [g], [R], params, T)
        corr, rep = csp.csp_propagate(ctx, g, p, params)
        torch.cuda.synchronize()
        assert rep.spmm_steps == 8
        assert np.max(np.abs(corr.cpu().numpy() - ref)) < 1e-10
    g.close()
