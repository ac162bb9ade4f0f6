"""The block contraction through LDS stages against the oracle: rows of odd
and even length (padded to 16 values), columns shorter and longer than a
workgroup's tiles, chunks of one, two and all steps of 16 orders, short last
blocks and the carried state."""
import numpy as np
import pytest
import torch

import oracle as o

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.mark.parametrize("kind,Lx,Ly,R,b,chunk", [
    ("square", 7, 5, 1, 32, 0),
    ("square", 37, 29, 3, 32, 0),
    ("square", 130, 61, 2, 32, 32),
    ("honeycomb", 19, 23, 5, 32, 48),
    ("honeycomb", 64, 40, 1, 8, 0),
    ("square", 48, 48, 3, 3, 16),
])
def test_states(csp, kind, Lx, Ly, R, b, chunk):
    print("[gpu] stages %s %dx%d R=%d b=%d chunk=%d" % (kind, Lx, Ly, R, b, chunk), flush=True)
    ctx = csp.Context(0)
    g = csp.Lattice(ctx, kind, Lx, Ly, t=-1.0, W=0.5, disorder_seed=3)
    c = o.Lattice(kind, Lx, Ly, t=-1.0, W=0.5, disorder_seed=3)
    psi = o.random_phase_states_fast(c.N, R, 9)
    Nt = 2 * b + (b + 1) // 2
    ref, _ = o.propagate(c, psi, Nt, b=0)
    p = torch.from_numpy(psi).to(torch.complex64).to("cuda:0")
    final = torch.empty_like(p)
    corr, _ = csp.csp_propagate(ctx, g, p, csp.make_params(
        Nt, mode="fp32_conc", block_b=b, chunk_K=chunk), final=final)
    torch.cuda.synchronize()
    # a product carries up to 3 * 2^-18 = 1.1e-5 of its value, the coefficients'
    # squares sum to about 1; 64 roundings of 2^-24 per carried block beside it
    assert np.max(np.abs(corr.cpu().numpy() - ref)) < 3e-5
    del g
    ctx.close()
