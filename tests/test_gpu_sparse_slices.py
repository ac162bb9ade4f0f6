"""Windowed explicit matrices at the sizes where their slices change form:
256 rows per slice (matrices of 160 MB and more), 128 rows, idle lanes at the
end of pocket slices, and tiles of unequal column counts.

On a periodic lattice without disorder a plane wave of momentum k is an
eigenstate, H psi = E(k) psi, so every value of the propagated state is known:
psi(t_j) = exp(-i pi j E / |H|) psi, and C_j = exp(-i pi j E / |H|)."""
import math

import numpy as np
import pytest
import torch

import csp_inputs as ci

pytestmark = pytest.mark.gpu

NT = 16


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.mark.parametrize("L,r_cut,R,mode,form", [
    (512, 6.1, 5, "fp32_conc", "moments"),   # 256 rows, no slice to spare
    (530, 6.1, 8, "fp32_conc", "states"),    # 256 rows, 4 + 4 columns, last slice short
    (530, 6.1, 3, "fp64_conc", "moments"),
    (331, 6.1, 7, "fp32_conc", "moments"),   # 128 rows, 3 + 2 + 2 columns
    (200, 3.0, 8, "fp64_conc", "states"),    # 3 + 3 + 2
    (97, 4.3, 1, "fp32_conc", "states"),
])
def test_plane_waves(csp, L, r_cut, R, mode, form):
    print("[gpu] slices L=%d r=%.1f R=%d %s %s" % (L, r_cut, R, mode, form), flush=True)
    ctx = csp.Context(0)
    col, val = ci.long_range_square(L, r_cut, t0=-1.0, decay=2.0, W=0.0, seed=1)
    lat = csp.Lattice.sparse(ctx, col, val)
    assert lat.info.ell_windowed == 1
    y, x = np.divmod(np.arange(L * L), L)
    E = np.empty(R)
    psi = np.empty((L * L, R), dtype=np.complex128)
    k = [(2 * math.pi * (3 * c + 1) / L, 2 * math.pi * (5 * c + 2) / L) for c in range(R)]
    # row 0 gives E(k): sum over its entries of H_0j e^{i k r_j}
    j0, v0 = np.asarray(col[0]), np.asarray(val[0], dtype=np.float64)
    use = j0 >= 0
    for c, (kx, ky) in enumerate(k):
        psi[:, c] = np.exp(1j * (kx * x + ky * y)) / L
        E[c] = np.sum(v0[use] * np.cos(kx * x[j0[use]] + ky * y[j0[use]]))
    dt = torch.complex64 if mode == "fp32_conc" else torch.complex128
    p = torch.from_numpy(psi).to(dt).to("cuda:0")
    par = csp.make_params(NT, mode=mode, block_b=8 if form == "states" else 0,
                          assembly=csp.CSP_ASSEMBLE_MOMENTS if form == "moments"
                          else csp.CSP_ASSEMBLE_STATES)
    final = torch.empty_like(p) if form == "states" else None
    corr, _ = csp.csp_propagate(ctx, lat, p, par, final=final)
    torch.cuda.synchronize()
    ph = np.exp(-1j * math.pi * np.arange(NT + 1)[:, None] * E[None, :] / lat.halfwidth)
    # about 110 orders, each a rounded sum of up to 121 terms: 110 * 2^-24 * 4
    # in complex64 (the split-bf16 assembly: 3 * 2^-18 beside it), and in
    # complex128 the same number of roundings of 2^-53 with room for the sums
    tol = 4e-5 if mode == "fp32_conc" else 1e-11
    assert np.max(np.abs(corr.cpu().numpy() - ph)) < tol
    if final is not None:
        assert np.max(np.abs(final.cpu().numpy() - psi * ph[-1])) * L < tol
    del lat
    ctx.close()
