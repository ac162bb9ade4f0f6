"""GPU: complex128 calls whose cap holds the workspace of four steps per launch
but not that of eight (a ring of 16 orders and eight more slots): they run
with four steps, or keep the chunk that four steps leave, with the results of
an uncapped call; and column windows of calls whose smallest workspace does not
fit for all columns at once.  Sums over other chunks and rows, in FP64: 1e-12 of values
of order one (correlations), of |psi|^2 = 1 (moments) and of the largest
element (quasi-eigenstates)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

L = 1024
VEC = L * L * 16           # one complex128 vector
MB = 1 << 20


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.fixture()
def ctx(csp):
    c = csp.Context(0)
    yield c
    c.close()


def lattice(csp, ctx):
    return csp.Lattice(ctx, "square", L, L, t=1.0, W=0.5, disorder_seed=3)


def state(R=1):
    gen = torch.Generator(device="cuda:0").manual_seed(7)
    ph = torch.rand((L * L, R), dtype=torch.float64, device="cuda:0", generator=gen) * (2 * np.pi)
    return torch.polar(torch.full_like(ph, 1.0 / L), ph)


@pytest.mark.parametrize("assembly,tuned,cap", [
    # 16 + kt slots, psi0, the carried state; tables and partial sums 66 MB
    (0, False, 23 * VEC + 66 * MB), (0, True, 23 * VEC + 66 * MB),
    # four slots and psi0; records of 4 and 8 steps: 9.4 and 21 MB
    (1, False, 5 * VEC + 15 * MB)])
def test_propagation_in_four_steps(csp, ctx, assembly, tuned, cap):
    print("[gpu] cap assembly=%d tuned=%d" % (assembly, tuned), flush=True)
    g, psi, Nt = lattice(csp, ctx), state(), 24
    ref, rep = csp.csp_propagate(ctx, g, psi, csp.make_params(Nt, mode="fp64_conc",
                                                              assembly=assembly))
    assert rep.spmm_steps == 8
    p = csp.make_params(Nt, mode="fp64_conc", assembly=assembly, mem_cap_bytes=cap)
    if tuned:
        T = csp.Tuning()
        T.spmm_vec, T.spmm_steps, T.spmm_seg_rows = 2, 8, 16
        T.contract_wg_per_cu, T.block_b = 4, 16
        csp.csp_set_tuning(ctx, [g], [1], p, T)
    ctx.trim()
    got, rep = csp.csp_propagate(ctx, g, psi, p)
    assert rep.spmm_steps == 4 and rep.n_passes == 1
    assert rep.workspace_bytes <= cap
    assert (got - ref).abs().max().item() < 1e-12
    # the least that four steps need is refused below it
    p = csp.make_params(Nt, mode="fp64_conc", assembly=assembly,
                        mem_cap_bytes=(21 * VEC + 64 * MB) if assembly == 0 else 5 * VEC)
    with pytest.raises(csp.CspError) as e:
        csp.csp_propagate(ctx, g, psi, p)
    assert e.value.status == csp.CSP_ENOMEM


@pytest.mark.parametrize("block,cap,K", [
    (0, 28, 16),        # 16 + kt slots, psi0, five accumulators: 26 and 30 vectors
    (0, 43, 32),        # 42 vectors with a chunk of 32 and four steps, 46 with eight
    (12, 54, 16)])      # forward and backward: 52 and 60
def test_quasi_eigenstates_in_four_steps(csp, ctx, block, cap, K):
    print("[gpu] cap qe block=%d" % block, flush=True)
    g, psi, Nt = lattice(csp, ctx), state(), 24
    E = [-2.0, -0.7, 0.1, 1.3, 2.2]
    ref, rep = csp.csp_quasi_eigenstates(ctx, g, psi, csp.make_params(
        Nt, mode="fp64_conc", block_b=block), E)
    assert rep.spmm_steps == 8
    ctx.trim()
    got, rep = csp.csp_quasi_eigenstates(ctx, g, psi, csp.make_params(
        Nt, mode="fp64_conc", block_b=block, mem_cap_bytes=cap * VEC), E)
    assert rep.spmm_steps == 4 and rep.chunk_K == K
    assert (got - ref).abs().max().item() < 1e-12 * ref.abs().max().item()


def test_conductivity_in_four_steps(csp, ctx):
    print("[gpu] cap ec", flush=True)
    g, psi, Nt = lattice(csp, ctx), state(), 24
    gen = torch.Generator(device="cuda:0").manual_seed(9)
    qe = torch.randn((5, L * L, 1), dtype=torch.complex128, device="cuda:0", generator=gen)
    ref, rep = csp.csp_ec_correlation(ctx, g, 0, psi, qe, csp.make_params(Nt, mode="fp64_conc"))
    assert rep.spmm_steps == 8
    ctx.trim()
    # 16 + kt slots, psi0, J psi, ten vectors of energies: 32 and 36
    got, rep = csp.csp_ec_correlation(ctx, g, 0, psi, qe, csp.make_params(
        Nt, mode="fp64_conc", mem_cap_bytes=34 * VEC))
    assert rep.spmm_steps == 4 and rep.chunk_K == 16
    assert (got - ref).abs().max().item() < 1e-12 * ref.abs().max().item()


@pytest.mark.parametrize("mode,slots,slack,passes,steps", [
    # two columns, one vector of both = 2 columns: 16 + kt slots, psi0, carry and
    # 66 MB of tables; complex64 at 8 steps 52 column vectors, complex128 at 4
    # steps 44, the sequential form 14 with neither tables nor a ring
    ("fp32_conc", 44, 98, 2, 8), ("fp64_conc", 40, 98, 2, 8), ("fp64_conc", 45, 67, 1, 4),
    ("fp64_seq", 20, 0, 1, 7), ("fp64_seq", 10, 0, 2, 7)])
def test_windows_by_the_real_need(csp, ctx, mode, slots, slack, passes, steps):
    print("[gpu] windows %s %d" % (mode, slots), flush=True)
    g, psi, Nt = lattice(csp, ctx), state(2), 6
    if mode == "fp32_conc":
        psi = psi.to(torch.complex64)
    ref, rep = csp.csp_propagate(ctx, g, psi, csp.make_params(Nt, mode=mode))
    assert rep.n_passes == 1
    cap = slots * (VEC // 2 if mode == "fp32_conc" else VEC) + slack * MB
    ctx.trim()
    got, rep = csp.csp_propagate(ctx, g, psi, csp.make_params(Nt, mode=mode, mem_cap_bytes=cap))
    assert rep.n_passes == passes and rep.spmm_steps == steps
    assert rep.workspace_bytes <= cap
    assert (got - ref).abs().max().item() < (2e-5 if mode == "fp32_conc" else 1e-12)
