"""GPU: the complex128 state kernel at eight steps per launch on the strip
forms' lattices (seams, open edges, short segments), and the contraction's two
complex64 kernels against each other."""
import numpy as np
import pytest

import csp_inputs as ci
import oracle as o
from test_gpu_strips import LATS

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


@pytest.mark.parametrize("spec", LATS)
def test_eight_step_states_match_oracle(csp, ctx, spec):
    """complex128 tolerance 1e-10, and five times that on the final states'
    largest element times sqrt(N)."""
    print("[gpu] fp64 strips %s %dx%d" % (spec["kind"], spec["Lx"], spec["Ly"]), flush=True)
    g = csp.Lattice(ctx, **spec)
    rest = {k: v for k, v in spec.items() if k not in ("kind", "Lx", "Ly", "center")}
    c = o.Lattice(spec["kind"], spec["Lx"], spec["Ly"], **rest)
    R, Nt, b = 2, 24, 9
    psi = o.random_phase_states_fast(c.N, R, 23)
    ref, _, fin_ref = o.propagate(c, psi, Nt, b=0, return_final=True, Hn=g.halfwidth,
                                  H0=spec.get("center", 0.0))
    p = torch.from_numpy(psi).to("cuda:0")
    for seg in (2, 8, 40):
        params = csp.make_params(Nt, mode="fp64_conc", block_b=b)
        T = csp.Tuning()
        T.spmm_vec, T.spmm_steps, T.spmm_seg_rows = 2, 8, seg
        T.contract_wg_per_cu, T.block_b = 4, b
        csp.csp_set_tuning(ctx, [g], [R], params, T)
        fin = torch.zeros_like(p)
        corr, rep = csp.csp_propagate(ctx, g, p, params, final=fin)
        torch.cuda.synchronize()
        assert rep.spmm_steps == 8
        assert np.max(np.abs(corr.cpu().numpy() - ref)) < 1e-10, seg
        assert np.max(np.abs(fin.cpu().numpy() - fin_ref)) * np.sqrt(c.N) < 5e-10, seg
    g.close()


@pytest.mark.parametrize("chunk", [0, 32, 48])
@pytest.mark.parametrize("b", [5, 20, 32])
def test_staged_contraction_is_the_register_form(csp, ctx, b, chunk):
    """Columns of an even number of values are contracted through LDS, odd ones
    from registers; both take the same operations in the same order.  The same
    matrix with one more, uncoupled site (its state zero) is odd: every
    correlation and every final value has the same bits."""
    print("[gpu] contraction forms b=%d K=%d" % (b, chunk), flush=True)
    L = 130                                          # 16900 sites: the last tile has 4
    col, val = ci.long_range_square(L, 3.0, t0=-1.0, decay=2.0, W=0.4, seed=5)
    N, R, Nt = L * L, 5, 2 * b + 3
    assert N % 2 == 0 and N % 32 != 0
    col1 = np.vstack([col, np.full((1, col.shape[1]), -1, dtype=col.dtype)])
    val1 = np.vstack([val, np.zeros((1, val.shape[1]), dtype=val.dtype)])
    psi = o.random_phase_states_fast(N, R, 6)
    out = []
    for cc, vv, n in ((col, val, N), (col1, val1, N + 1)):
        g = csp.Lattice.sparse(ctx, cc, vv)
        p = torch.zeros((n, R), dtype=torch.complex64, device="cuda:0")
        p[:N] = torch.from_numpy(psi).to("cuda:0")
        fin = torch.zeros_like(p)
        corr, rep = csp.csp_propagate(ctx, g, p, csp.make_params(
            Nt, mode="fp32_conc", block_b=b, chunk_K=chunk), final=fin)
        torch.cuda.synchronize()
        out.append((g.halfwidth, corr, fin[:N].clone(), rep.chunk_K))
        g.close()
    assert out[0][0] == out[1][0] and out[0][3] == out[1][3]
    # (C_0 is a sum over all sites in other groups)
    assert torch.equal(out[0][1][1:], out[1][1][1:])
    assert torch.equal(out[0][2], out[1][2])
