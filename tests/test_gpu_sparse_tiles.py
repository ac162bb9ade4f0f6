"""Windowed explicit matrices in the wide tiles: 4 to 8 columns a workgroup in
complex64, 4 to 7 in complex128 (6 and 7 with 64 to 78 KB of LDS), slices of 128
and 256 rows, every form.

On a periodic lattice without disorder a plane wave of momentum k is an
eigenstate, H psi = E(k) psi, so every value of the propagated state is known:
psi(t_j) = exp(-i pi j E / |H|) psi, and C_j = exp(-i pi j E / |H|)."""
import math

import numpy as np
import pytest

import csp_inputs as ci

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NT = 16


@pytest.fixture(scope="module")
def csp():
    import paper_2510_17432_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(csp):
    c = csp.Context(0)
    yield c
    c.close()


_lat = {}


def lattice(csp, ctx, L, r_cut):
    if (L, r_cut) not in _lat:
        _lat.clear()
        col, val = ci.long_range_square(L, r_cut, t0=-1.0, decay=2.0, W=0.0, seed=1)
        _lat[(L, r_cut)] = (csp.Lattice.sparse(ctx, col, val), np.asarray(col[0]),
                            np.asarray(val[0], dtype=np.float64))
    return _lat[(L, r_cut)]


@pytest.mark.parametrize("L,r_cut,mode,columns", [
    (400, 4.3, "fp32_conc", (5, 7, 8)),       # 128 rows: 5, 7 and 3 + 3 + 2 (states 4 + 4)
    (300, 6.1, "fp32_conc", (8, 10)),         # 4 + 4, 5 + 5
    (450, 8.6, "fp32_conc", (6, 7, 8)),       # a matrix of 270 MB, 128 rows: 6, 7, 8
    (530, 6.1, "fp32_conc", (7, 12)),         # 256 rows: 7, 4 + 4 + 4
    (300, 6.1, "fp64_conc", (4, 5, 6, 8)),    # 128 rows: 4, 5, 3 + 3 (states 6), 4 + 4
    (530, 6.1, "fp64_conc", (6, 9)),          # 256 rows: 6 (78 KB of LDS), 5 + 4
    (720, 4.3, "fp64_conc", (7,)),            # 256 rows: 7
])
@pytest.mark.parametrize("form", ["moments", "blocks", "states"])
def test_plane_waves_in_wide_tiles(csp, ctx, L, r_cut, mode, columns, form):
    lat, j0, v0 = lattice(csp, ctx, L, r_cut)
    assert lat.info.ell_windowed == 1
    y, x = np.divmod(np.arange(L * L), L)
    use = j0 >= 0
    for R in columns:
        print("[gpu] tiles L=%d r=%.1f R=%d %s %s" % (L, r_cut, R, mode, form), flush=True)
        E = np.empty(R)
        psi = np.empty((L * L, R), dtype=np.complex128)
        for c in range(R):
            kx, ky = 2 * math.pi * (3 * c + 1) / L, 2 * math.pi * (5 * c + 2) / L
            psi[:, c] = np.exp(1j * (kx * x + ky * y)) / L
            E[c] = np.sum(v0[use] * np.cos(kx * x[j0[use]] + ky * y[j0[use]]))
        dt = torch.complex64 if mode == "fp32_conc" else torch.complex128
        p = torch.from_numpy(psi).to(dt).to("cuda:0")
        par = csp.make_params(NT, mode=mode, block_b=0 if form == "moments" else 8,
                              assembly=csp.CSP_ASSEMBLE_STATES if form == "states"
                              else csp.CSP_ASSEMBLE_MOMENTS)
        final = None if form == "moments" else torch.empty_like(p)
        corr, _ = csp.csp_propagate(ctx, lat, p, par, final=final)
        torch.cuda.synchronize()
        ph = np.exp(-1j * math.pi * np.arange(NT + 1)[:, None] * E[None, :] / lat.halfwidth)
        # about 110 orders, each a rounded sum of up to 233 terms: 110 * 2^-24 * 4
        # in complex64 (the split-bf16 assembly: 3 * 2^-18 beside it), and in
        # complex128 the same number of roundings of 2^-53 with room for the sums
        tol = 4e-5 if mode == "fp32_conc" else 1e-11
        assert np.max(np.abs(corr.cpu().numpy() - ph)) < tol
        if final is not None:
            assert np.max(np.abs(final.cpu().numpy() - psi * ph[-1])) * L < tol
