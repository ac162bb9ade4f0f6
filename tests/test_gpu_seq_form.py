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
