"""GPU: the sequential complex128 form of stencil lattices beside tuning
records, in a batch, and in column windows.  complex128 sums in another order
than the oracle's or the other call's: 1e-10 and 1e-12."""
import numpy as np
import pytest

import oracle as o

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.fixture()
def ctx(csp):
    c = csp.Context(0)
    yield c
    c.close()


def test_tuning_records_do_not_shape_the_sequential_kernel(csp, ctx):
    # a record's rows per work item were measured on the ring's kernel; one row
    # per item shows in the workspace of the step sums
    g = csp.Lattice(ctx, "square", 512, 256, t=1.0, W=0.4, disorder_seed=1)
    psi = torch.from_numpy(o.random_phase_states_fast(512 * 256, 2, 3)).to("cuda:0")
    p = csp.make_params(5, mode="fp64_seq")
    ref, rep = csp.csp_propagate(ctx, g, psi, p)
    T = csp.Tuning()
    T.spmm_vec, T.spmm_steps, T.spmm_seg_rows = 2, 4, 1
    T.contract_wg_per_cu, T.block_b = 4, 1
    csp.csp_set_tuning(ctx, [g], [2], p, T)
    ctx.trim()
    got, rep2 = csp.csp_propagate(ctx, g, psi, p)
    assert rep2.contract_launches == 0
    assert rep2.workspace_bytes == rep.workspace_bytes
    assert torch.equal(got, ref)
    g.close()


@pytest.mark.parametrize("graph", [-1, 0])
def test_sequential_batch(csp, ctx, graph):
    # several lattices of both kinds in one call, odd column counts (groups of
    # 2 and 1) and more steps than the records of one sum; without graph replay
    # the recursion accumulates the states, with it the ring does
    specs = [dict(kind="square", Lx=97, Ly=61, t=1.0, W=0.6, disorder_seed=4),
             dict(kind="honeycomb", Lx=40, Ly=33, t=-2.7, W=0.0, periodic_y=False),
             dict(kind="square", Lx=250, Ly=5, t=-1.0, W=0.0),
             dict(kind="honeycomb", Lx=90, Ly=70, t=-2.7, W=1.0, disorder_seed=6),
             dict(kind="chain", Lx=333, Ly=1, t=1.0, W=0.2, disorder_seed=8)]
    Nt, lats, psis, refs = 19, [], [], []
    for i, spec in enumerate(specs):
        g = csp.Lattice(ctx, **spec)
        rest = {k: v for k, v in spec.items() if k not in ("kind", "Lx", "Ly")}
        c = o.Lattice(spec["kind"], spec["Lx"], spec["Ly"], **rest)
        psi = o.random_phase_states_fast(c.N, 1 + i % 3, 40 + i)
        refs.append(o.propagate(c, psi, Nt, b=0, Hn=g.halfwidth)[0])
        lats.append(g)
        psis.append(torch.from_numpy(psi).to("cuda:0"))
    got, rep = csp.csp_propagate_batch(ctx, lats, psis, csp.make_params(
        Nt, mode="fp64_seq", graph=graph))
    torch.cuda.synchronize()
    assert (rep.contract_launches == 0) == (graph == -1)
    for ref, x in zip(refs, got):
        assert np.max(np.abs(x.cpu().numpy() - ref)) < 1e-10
    for g in lats:
        g.close()
