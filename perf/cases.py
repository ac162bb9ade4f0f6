"""The work that programs have this library do, as measurable cases.

listed() names twelve of them, from a 64 x 64 lattice whose call is over in
milliseconds to 2.7e8 orbitals; draw(rng) gives more of the same ranges.
prepare() makes what a program holds before the call (lattice or explicit
matrix, state block, energies), run() is one pass through the public entry
points, exact() the same results from plain torch in 64 bits, and work() the
bytes and operations that no implementation can do without.

Forms (the key "form"):
  moments     csp_propagate, CSP_ASSEMBLE_MOMENTS, one block (the DOS), then csp_dos
  mom_blocks  csp_propagate, CSP_ASSEMBLE_MOMENTS in time blocks, with the final states
  states      csp_propagate, CSP_ASSEMBLE_STATES (or the sequential complex128 mode)
  batch       csp_propagate_batch over lattices of uneven sizes
  qe          csp_quasi_eigenstates (block 0: energy-based, >= 1: state-based)
  ec          csp_ec_correlation and csp_ec_sigma
"""
import functools
import math
import random

import numpy as np
import torch

import csp_inputs
import paper_2510_17432_amd as csp

DEV = "cuda:0"
PI = math.pi


def _case(name, form, kind, Lx, Ly, t, W, R, Nt, mode="fp32_conc", block=0, chunk=0, sites=0,
          final=False, n_E=0, r_cut=0.0, count=1, periodic=True):
    c = dict(form=form, kind=kind, Lx=Lx, Ly=Ly, t=t, W=W, R=R, Nt=Nt, mode=mode, block=block,
             chunk=chunk, sites=sites, final=final, n_E=n_E, r_cut=r_cut, count=count,
             periodic=periodic)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The first thing a new user runs, and one sample of a disorder
        # average over many small lattices: DOS of the 64 x 64 square lattice.
        _case("dos_square64", "moments", "square", 64, 64, 1.0, 0.0, 1, 1024),
        # The same lattice propagated state by state in time blocks of the
        # library's choice, the final state kept for the next stage.
        _case("states_square64", "states", "square", 64, 64, 1.0, 0.0, 1, 1024, final=True),
        # DOS of graphene (2.1 M orbitals, 4 random-phase columns) over the
        # full 2048 steps: the ordinary production call.
        _case("dos_graphene", "moments", "honeycomb", 1024, 1024, -2.7, 0.0, 4, 2048),
        # DOS and LDOS of graphene together: 64 localized states beside the
        # random ones; two time blocks of the state assembly.
        _case("ldos_graphene", "states", "honeycomb", 1024, 1024, -2.7, 0.0, 4, 64, block=32,
              sites=64),
        # A disordered lattice of odd side (unaligned rows) and three columns
        # (groups of 2 and 1), final states kept, a last block that is short.
        _case("states_square4099", "states", "square", 4099, 4099, 1.0, 0.5, 3, 80, block=32,
              final=True),
        # One time block of a lattice whose vectors fill the card: the
        # contraction runs in chunks of 16 orders, as at 31623^2 orbitals.
        _case("states_square16383", "states", "square", 16383, 16383, 1.0, 0.5, 2, 32, block=32,
              chunk=16),
        # The plain sequential complex128 form that results are checked
        # against, with its final states.
        _case("sequential_graphene", "states", "honeycomb", 1024, 1024, -2.7, 0.0, 4, 24,
              mode="fp64_seq", final=True),
        # The complex128 reference DOS of a disordered lattice.
        _case("dos_fp64_square2047", "moments", "square", 2047, 2047, 1.0, 0.5, 4, 512,
              mode="fp64_conc"),
        # Disorder and size average: uneven lattices of both kinds in one call.
        _case("batch_uneven", "batch", "square", 512, 512, 1.0, 1.0, 8, 256, count=16),
        # An explicit Hamiltonian of matrix density 121 (long-range hopping),
        # 5 random-phase columns: the DOS of a dense tight-binding model.
        _case("dos_explicit121", "moments", "long_range", 512, 512, -1.0, 0.5, 5, 384,
              r_cut=6.1),
        # Quasi-eigenstates at 49 energies, the input of the conductivity.
        _case("qe_graphene512", "qe", "honeycomb", 512, 512, -2.7, 0.0, 2, 512, n_E=49),
        # Conductivity of disordered graphene at 49 energies, complex128.
        _case("ec_fp64_graphene256", "ec", "honeycomb", 256, 256, -2.7, 1.0, 2, 512,
              mode="fp64_conc", n_E=49),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choice(["moments", "moments", "states", "states", "states", "mom_blocks", "batch",
                       "qe", "ec", "explicit"])
    r_cut = 0.0
    if form == "explicit":
        form = rng.choice(["moments", "states"])
        kind, r_cut = "long_range", rng.choice([3.0, 4.3, 6.1])
        Lx = Ly = _log_int(rng, 40, 480)
    else:
        kind = rng.choice(["square", "honeycomb"])
        top = {"moments": 4096, "states": 4096, "mom_blocks": 2048, "batch": 400, "qe": 500,
               "ec": 300}[form]
        Lx, Ly = _log_int(rng, 48, top), _log_int(rng, 48, top)
        if kind == "honeycomb":
            Lx = max(24, Lx // 2)
    mode = "fp32_conc"
    if form in ("moments", "ec", "qe", "mom_blocks"):
        mode = rng.choice(["fp32_conc", "fp32_conc", "fp64_conc"])
    elif form == "states":
        mode = rng.choice(["fp32_conc", "fp32_conc", "fp64_conc", "fp64_seq"])
    R = rng.randint(1, 4) if form in ("qe", "ec") else rng.randint(1, 9)
    n_orb = Lx * Ly * (2 if kind == "honeycomb" else 1)
    heavy = n_orb * R * (2 if mode != "fp32_conc" else 1)
    if kind == "long_range":
        heavy *= 12
    # time steps: many on small lattices, few on the largest
    most = max(24, min(1500, int(6e9 / heavy)))
    if form in ("states", "mom_blocks"):
        most = max(16, most // 6)
    Nt = _log_int(rng, 16, most)
    n_E = block = 0
    if form in ("qe", "ec"):
        n_E = rng.choice([5, 12, 31, 49])
        Nt = min(Nt, 500)
        if form == "qe" and n_E <= (15 if mode == "fp64_conc" else 31) and rng.random() < 0.4:
            block = rng.randint(8, 40)
    elif form == "mom_blocks":
        block = rng.randint(8, 64)
    elif form == "states" and mode == "fp32_conc":
        block = rng.choice([0, 7, 16, 32, 45])
    count = rng.randint(3, 14) if form == "batch" else 1
    W = rng.choice([0.0, 0.5, 1.0])
    t = -1.0 if kind == "long_range" else (1.0 if kind == "square" else -2.7)
    final = form == "mom_blocks" or (form == "states" and rng.random() < 0.5)
    periodic = kind == "long_range" or rng.random() < 0.8
    return _case(None, form, kind, Lx, Ly, t, W, R, Nt, mode=mode, block=block, final=final,
                 n_E=n_E, r_cut=r_cut, count=count, periodic=periodic)


# ------------------------------------------------------------------ inputs
def _members(case):
    """The lattices of a case: one, or those of a batch (both kinds, uneven
    sizes and column counts, drawn from the sizes of the case)."""
    if case["form"] != "batch":
        return [case]
    rng = random.Random(7 * case["Lx"] + case["count"])
    out = []
    for i in range(case["count"]):
        kind = ("square", "honeycomb")[i % 2]
        side = _log_int(rng, min(64, case["Lx"]), case["Lx"])
        out.append(dict(case, kind=kind, Lx=side, Ly=max(24, _log_int(rng, side // 2, side)),
                        t=1.0 if kind == "square" else -2.7, W=case["W"] * rng.random(),
                        R=rng.randint(1, case["R"])))
    return out


def _orbitals(m):
    return m["Lx"] * m["Ly"] * (2 if m["kind"] == "honeycomb" else 1)


def _columns(m):
    return m["R"] + m["sites"]


def _dtype(m):
    return torch.complex64 if m["mode"] == "fp32_conc" else torch.complex128


def _states(m, seed):
    """Random-phase columns (norm 1), then unit vectors at random sites."""
    N = _orbitals(m)
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1) + 17)
    psi = torch.empty((N, _columns(m)), dtype=_dtype(m), device=DEV)
    for r in range(m["R"]):
        ph = torch.rand(N, dtype=torch.float64, device=DEV, generator=g) * (2.0 * PI)
        psi[:, r] = torch.polar(torch.full_like(ph, 1.0 / math.sqrt(N)), ph)
    if m["sites"]:
        psi[:, m["R"]:] = 0
        at = torch.randperm(N, device=DEV, generator=g)[:m["sites"]]
        psi[at, m["R"] + torch.arange(m["sites"], device=DEV)] = 1
    return psi


def _disorder_seed(seed, i):
    return 1000 * (seed + 1) + i


@functools.lru_cache(maxsize=4)
def _long_range(L, r_cut, t, W, seed):
    return csp_inputs.long_range_square(L, r_cut, t0=t, decay=2.0, W=W, seed=seed)


_CTX = []


def _context():
    """A program keeps one context (stream, workspace) for all its calls."""
    if not _CTX:
        _CTX.append(csp.Context(0))
    return _CTX[0]


def _energies(m):
    """n_E energies across the band."""
    half = 0.7 * (3 if m["kind"] == "honeycomb" else 4) * abs(m["t"])
    return [half * (2.0 * (e + 0.5) / m["n_E"] - 1.0) for e in range(m["n_E"])]


def prepare(case, seed):
    ctx = _context()
    s = {"ctx": ctx, "form": case["form"], "lats": [], "psi": []}
    members = _members(case)
    for i, m in enumerate(members):
        if m["kind"] == "long_range":
            col, val = _long_range(m["Lx"], m["r_cut"], m["t"], m["W"], _disorder_seed(seed, i))
            lat = csp.Lattice.sparse(ctx, col, val)
        else:
            lat = csp.Lattice(ctx, m["kind"], m["Lx"], m["Ly"], t=m["t"], W=m["W"],
                              disorder_seed=_disorder_seed(seed, i), periodic_x=m["periodic"],
                              periodic_y=m["periodic"])
        s["lats"].append(lat)
        s["psi"].append(_states(m, seed + 31 * i))
    m = members[0]
    moments = case["form"] in ("moments", "mom_blocks")
    s["params"] = csp.make_params(
        case["Nt"], mode=case["mode"], block_b=case["block"], chunk_K=case["chunk"],
        assembly=csp.CSP_ASSEMBLE_MOMENTS if moments else csp.CSP_ASSEMBLE_STATES)
    s["final"] = bool(case["final"])
    if case["n_E"]:
        s["energies"] = _energies(m)
    if case["form"] == "ec":
        s["qe"] = _quasi_eigenstates(m, seed, 96).to(_dtype(m))
    return s


def run(s):
    ctx, p = s["ctx"], s["params"]
    if s["form"] == "batch":
        return csp.csp_propagate_batch(ctx, s["lats"], s["psi"], p)[0]
    lat, psi = s["lats"][0], s["psi"][0]
    if s["form"] == "qe":
        return csp.csp_quasi_eigenstates(ctx, lat, psi, p, s["energies"])[0]
    if s["form"] == "ec":
        corr, _ = csp.csp_ec_correlation(ctx, lat, 0, psi, s["qe"], p)
        sigma = csp.csp_ec_sigma(ctx, corr, lat.halfwidth, s["energies"])
        return {"corr": corr, "sigma": sigma}
    final = torch.empty_like(psi) if s["final"] else None
    corr, _ = csp.csp_propagate(ctx, lat, psi, p, final=final)
    out = {"corr": corr}
    if final is not None:
        out["final"] = final
    if s["form"] == "moments":
        out["E"], out["D"], out["D_mean"] = csp.csp_dos(ctx, corr, lat.halfwidth,
                                                        center=lat.info.H0)
    return out


# ------------------------------------------------------------------ work
def _order(x):
    """Chebyshev order of exp(-i x y) to 1e-14."""
    M = 1 << int(math.ceil(math.log2(2.0 * x + 200.0)))
    th = 2.0 * PI * np.arange(M) / M
    c = np.abs(np.fft.fft(np.exp(-1j * x * np.cos(th)))[:M // 2]) * (2.0 / M)
    n = int(math.floor(x)) + 1
    while n < M // 2 - 1 and c[n] > 1e-14:
        n += 1
    return n


def _degree(m):
    if m["kind"] == "long_range":
        R = int(m["r_cut"])
        return sum(0 < dx * dx + dy * dy <= m["r_cut"] ** 2
                   for dx in range(-R, R + 1) for dy in range(-R, R + 1))
    return 4 if m["kind"] == "square" else 3


def work(case):
    """Bytes: the states and on-site energies (or the matrix) read once, the
    outputs written once.  Operations: the recursion (2 per neighbour and
    component, scale and subtract, on-site term) of every Chebyshev step of
    the form and the sums that the form takes over the orders."""
    nbytes = flops = 0.0
    for m in _members(case):
        N, R, Nt = _orbitals(m), _columns(m), m["Nt"]
        v = N * R
        csz = 8 if m["mode"] == "fp32_conc" else 16
        deg = _degree(m)
        step = (4 * deg if m["kind"] == "long_range" else 2 * deg) + 4 + (4 if m["W"] else 0)
        nbytes += v * csz + 16.0 * (Nt + 1) * R
        if m["kind"] == "long_range":
            nbytes += N * (deg + 1) * (4 + csz // 2)
        elif m["W"]:
            nbytes += N * csz // 2
        if case["form"] == "moments":
            n = (_order(Nt * PI) + 1) // 2
            flops += v * n * (step + 8.0)
            flops += 4.0 * Nt * n * R
        elif case["form"] in ("states", "batch", "mom_blocks"):
            b = 1 if m["mode"] == "fp64_seq" else (m["block"] or 32)
            b = min(b, Nt, 16 if m["mode"] == "fp64_conc" and case["form"] == "states" else Nt)
            blocks, last = divmod(Nt, b)
            for k, cnt in ((b, blocks), (last, 1 if last else 0)):
                if cnt:
                    n = _order(k * PI)
                    # a real coefficient per order and time (states), or a
                    # moment per order and the carried state
                    sums = 4.0 * k if case["form"] != "mom_blocks" else 12.0
                    flops += cnt * v * (n * (step + sums) + 8.0 * k)
            if m["final"]:
                nbytes += v * csz
        else:
            n = _order(Nt * PI)
            nbytes += float(v) * m["n_E"] * csz
            flops += v * n * (step + (4.0 if case["form"] == "qe" else 8.0) * m["n_E"])
            if case["form"] == "ec":
                nbytes += 16.0 * (Nt + 1) * R * m["n_E"]
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ 64-bit results
# Plain torch: the Hamiltonian by shifted copies (or by FFT where the hopping
# is a translation-invariant kernel), functions of it by Chebyshev sums whose
# coefficients come from the quadrature of cos(n theta) on a cosine grid.
def _onsite(N, W, seed):
    """W (u_s - 1/2), u_s the SplitMix64 draw s of the seed, top 53 bits."""
    def mul(x, k):
        return x * (k - (1 << 64) if k >> 63 else k)

    def shr(x, k):
        return (x >> k) & ((1 << (64 - k)) - 1)

    z = mul(torch.arange(1, N + 1, dtype=torch.int64, device=DEV), 0x9e3779b97f4a7c15) + seed
    z = mul(z ^ shr(z, 30), 0xbf58476d1ce4e5b9)
    z = mul(z ^ shr(z, 27), 0x94d049bb133111eb)
    z ^= shr(z, 31)
    return W * (shr(z, 11).to(torch.float64) * 2.0 ** -53 - 0.5)


class _H:
    """H and its half-width in 64 bits; apply() takes [N][R] blocks."""

    def __init__(self, m, seed, i=0):
        self.m = m
        N, Lx, Ly = _orbitals(m), m["Lx"], m["Ly"]
        ds = _disorder_seed(seed, i)
        if m["kind"] == "long_range":
            R = int(m["r_cut"])
            ker = torch.zeros((Ly, Lx), dtype=torch.float64)
            for dx in range(-R, R + 1):
                for dy in range(-R, R + 1):
                    d2 = dx * dx + dy * dy
                    if 0 < d2 <= m["r_cut"] ** 2:
                        ker[dy % Ly, dx % Lx] += m["t"] * math.exp(-(math.sqrt(d2) - 1.0) / 2.0)
            self.ker = torch.fft.fft2(ker.to(DEV)).reshape(Ly, Lx, 1)
            eps = m["W"] * (np.random.default_rng(ds).random(N) - 0.5) if m["W"] else np.zeros(N)
            self.eps = torch.from_numpy(eps).to(DEV)
            hop = ker.abs().sum().item()
            top = float(self.eps.abs().max()) + hop
        else:
            self.eps = _onsite(N, m["W"], ds) if m["W"] else None
            deg = self.hop(torch.ones((N, 1), dtype=torch.float64, device=DEV)).abs()[:, 0]
            top = float((deg if self.eps is None else deg + self.eps.abs()).max())
        self.half = 1.025 * top

    def _shift(self, x, by, axis):
        """Neighbour values: y[k] = x[k - by], zero past an open edge."""
        y = torch.roll(x, by, axis)
        if not self.m["periodic"]:
            y.select(axis, 0 if by > 0 else -1).zero_()
        return y

    def hop(self, x):
        m, R = self.m, x.shape[1]
        if m["kind"] == "square":
            g = x.reshape(m["Ly"], m["Lx"], R)
            y = self._shift(g, 1, 0)
            for by, ax in ((-1, 0), (1, 1), (-1, 1)):
                y += self._shift(g, by, ax)
            return y.reshape(-1, R).mul_(m["t"])
        g = x.reshape(m["Ly"], m["Lx"], 2, R)
        A, B = g[:, :, 0], g[:, :, 1]
        a = B + self._shift(B, 1, 1) + self._shift(B, 1, 0)
        b = A + self._shift(A, -1, 1) + self._shift(A, -1, 0)
        return torch.stack((a, b), 2).reshape(-1, R).mul_(m["t"])

    def scaled(self, x):
        """H x / |H|."""
        m = self.m
        if m["kind"] == "long_range":
            g = torch.fft.fft2(x.reshape(m["Ly"], m["Lx"], -1), dim=(0, 1))
            y = torch.fft.ifft2(g * self.ker, dim=(0, 1)).reshape(x.shape)
        else:
            y = self.hop(x)
        if self.eps is not None:
            y += self.eps[:, None] * x
        return y.div_(self.half)

    def current_x(self, x):
        """i [H, X] x of the nearest-neighbour lattices (bond lengths 1)."""
        m, R = self.m, x.shape[1]
        if m["kind"] == "square":
            g = x.reshape(m["Ly"], m["Lx"], R)
            y = self._shift(g, -1, 1) - self._shift(g, 1, 1)
            return (1j * m["t"]) * y.reshape(-1, R)
        g = x.reshape(m["Ly"], m["Lx"], 2, R)
        A, B, h = g[:, :, 0], g[:, :, 1], math.sqrt(3.0) / 2.0
        a = (B - self._shift(B, 1, 1)) * h
        b = (self._shift(A, -1, 1) - A) * h
        return (1j * m["t"]) * torch.stack((a, b), 2).reshape(-1, R)

    def vectors(self, x, n):
        """T_0 x .. T_n x, one after another."""
        p, c = x, self.scaled(x)
        yield p
        if n >= 1:
            yield c
        for _ in range(2, n + 1):
            q = self.scaled(c)
            p = q.mul_(2.0).sub_(p)
            p, c = c, p
            yield c


def _dot(a, b):
    """<a_r|b_r> per column."""
    return (a.conj() * b).sum(0)


def _grid(n):
    M = 1 << int(math.ceil(math.log2(2.0 * n + 64.0)))
    return (torch.arange(M, dtype=torch.float64, device=DEV) + 0.5) * (PI / M)


def _cheb_coeffs(f, n):
    """Chebyshev coefficients 0..n of the functions f [rows][M] on _grid(n)."""
    th = _grid(n)
    out = torch.empty((f.shape[0], n + 1), dtype=f.dtype, device=DEV)
    for lo in range(0, n + 1, 512):
        k = torch.arange(lo, min(lo + 512, n + 1), dtype=torch.float64, device=DEV)
        c = torch.cos(th[:, None] * k[None, :]).to(f.dtype)
        out[:, lo:lo + 512] = (f @ c) * (2.0 / th.numel())
    out[:, 0] *= 0.5
    return out


def _from_moments(mom, Nt, sign=-1.0):
    """sum_n c_n(j pi) m_n for j = 0..Nt: mom [n + 1][cols] -> [Nt + 1][cols]."""
    n = mom.shape[0] - 1
    th = _grid(n)
    g = torch.zeros((th.numel(), mom.shape[1]), dtype=torch.complex128, device=DEV)
    for lo in range(0, n + 1, 512):
        k = torch.arange(lo, min(lo + 512, n + 1), dtype=torch.float64, device=DEV)
        c = torch.cos(th[:, None] * k[None, :])
        c *= torch.where(k == 0, 1.0, 2.0)
        g += c.to(torch.complex128) @ mom[lo:lo + 512]
    y = torch.cos(th)
    out = torch.empty((Nt + 1, mom.shape[1]), dtype=torch.complex128, device=DEV)
    for lo in range(0, Nt + 1, 256):
        x = torch.arange(lo, min(lo + 256, Nt + 1), dtype=torch.float64, device=DEV) * PI
        ph = x[:, None] * y[None, :]
        out[lo:lo + 256] = torch.polar(torch.ones_like(ph), sign * ph) @ g / th.numel()
    return out


def _correlations(H, psi, Nt):
    """<psi|exp(-i H~ j pi)|psi>, the moments by the product identity."""
    n = _order(Nt * PI)
    mom = torch.zeros((n + 2, psi.shape[1]), dtype=torch.complex128, device=DEV)
    prev = None
    for k, v in enumerate(H.vectors(psi, n // 2 + 1)):
        if 2 * k <= n:
            mom[2 * k] = 2.0 * _dot(v, v) - mom[0] if k else _dot(v, v)
        if k and 2 * k - 1 <= n:
            mom[2 * k - 1] = 2.0 * _dot(v, prev) - mom[1] if k > 1 else _dot(v, prev)
        prev = v
    return _from_moments(mom[:n + 1], Nt)


def _final(H, psi, Nt):
    n = _order(Nt * PI)
    f = torch.polar(torch.ones_like(_grid(n)), -Nt * PI * torch.cos(_grid(n)))[None, :]
    c = _cheb_coeffs(f, n)[0].tolist()
    out = torch.zeros_like(psi)
    for k, v in enumerate(H.vectors(psi, n)):
        out += c[k] * v
    return out


def _filter(H, psi, energies, Nt):
    """tau sum_j (2 - delta_j0) cos(E t_j - x_j H~) psi at every energy: [n_E][N][R]."""
    tau = PI / H.half
    n = _order(Nt * PI)
    y = torch.cos(_grid(n))
    f = torch.full((len(energies), y.numel()), 1.0, dtype=torch.float64, device=DEV)
    E = torch.tensor(energies, dtype=torch.float64, device=DEV)
    z = E[:, None] * tau - PI * y[None, :]
    for j in range(1, Nt + 1):
        f += 2.0 * torch.cos(j * z)
    c = _cheb_coeffs(f * tau, n).to(torch.complex128)
    out = torch.zeros((len(energies), psi.numel()), dtype=torch.complex128, device=DEV)
    buf = []
    k0 = 0
    for k, v in enumerate(H.vectors(psi, n)):
        buf.append(v.reshape(-1).clone())
        if len(buf) == 32 or k == n:
            out += c[:, k0:k + 1] @ torch.stack(buf)
            buf, k0 = [], k + 1
    return out.reshape(len(energies), *psi.shape)


def _quasi_eigenstates(m, seed, Nt):
    """Quasi-eigenstates as a program has them before the conductivity."""
    psi = _states(m, seed).to(torch.complex128)
    return _filter(_H(m, seed), psi, _energies(m), Nt)


def _too_long(case):
    per = 6.0 if case["kind"] == "long_range" else 1.0
    if case["form"] in ("states", "mom_blocks"):
        per *= 2.5 if case["final"] else 1.0
    if case["form"] in ("qe", "ec"):
        per *= 2.0 + case["n_E"] / 8.0
    vals = sum(_orbitals(m) * _columns(m) for m in _members(case))
    return vals * per * _order(case["Nt"] * PI) > 1.5e11


def exact(case, seed):
    if _too_long(case):
        return None
    if case["form"] == "batch":
        return [_correlations(_H(m, seed, i), _states(m, seed + 31 * i).to(torch.complex128),
                              m["Nt"]) for i, m in enumerate(_members(case))]
    H = _H(case, seed)
    psi = _states(case, seed)
    Nt = case["Nt"]
    if case["form"] == "qe":
        return _filter(H, psi.to(torch.complex128), _energies(case), Nt)
    if case["form"] == "ec":
        psi = psi.to(torch.complex128)
        qe = _quasi_eigenstates(case, seed, 96).to(_dtype(case)).to(torch.complex128)
        n_E, N, R = qe.shape
        n = _order(Nt * PI)
        corr = torch.empty((n_E, Nt + 1, R), dtype=torch.complex128, device=DEV)
        for r in range(R):
            bra = torch.stack([H.current_x(qe[e, :, r:r + 1])[:, 0] for e in range(n_E)])
            bra = bra.conj().resolve_conj()
            mom = torch.empty((n + 1, n_E), dtype=torch.complex128, device=DEV)
            for k, v in enumerate(H.vectors(H.current_x(psi[:, r:r + 1]), n)):
                mom[k] = torch.mv(bra, v[:, 0])
            norm = (psi[:, r].conj()[None, :] * qe[:, :, r]).sum(1).abs()
            # <J psi|T_n|J Psi> is the conjugate of the sums above
            corr[:, :, r] = (_from_moments(mom, Nt).conj() / norm[None, :]).T
        tau = PI / H.half
        tj = torch.arange(Nt + 1, dtype=torch.float64, device=DEV) * tau
        w = torch.full_like(tj, tau)
        w[0] = w[-1] = tau / 2.0
        E = torch.tensor(_energies(case), dtype=torch.float64, device=DEV)
        ph = torch.polar(w[None, :].expand(n_E, -1).contiguous(), -E[:, None] * tj[None, :])
        return {"corr": corr, "sigma": (ph[:, :, None] * corr).sum(1).real}
    cols = []
    for r in range(psi.shape[1]):        # one column at a time: the largest fill the card
        cols.append(_correlations(H, psi[:, r:r + 1].to(torch.complex128), Nt))
    out = {"corr": torch.cat(cols, 1)}
    if case["final"]:
        out["final"] = torch.cat([_final(H, psi[:, r:r + 1].to(torch.complex128), Nt)
                                  for r in range(psi.shape[1])], 1)
    if case["form"] == "moments":
        tau = PI / H.half
        C = out["corr"]
        j = torch.arange(Nt + 1, dtype=torch.float64, device=DEV)
        w = 0.5 * (1.0 + torch.cos(PI * j / Nt))
        full = torch.zeros((2 * Nt, C.shape[1]), dtype=torch.complex128, device=DEV)
        full[:Nt] = w[:Nt, None] * C[:Nt]
        full[Nt + 1:] = (w[1:Nt, None] * C[1:Nt].conj()).flip(0)
        full[Nt] = w[Nt] * C[Nt].conj()
        D = torch.fft.fftshift(torch.fft.ifft(full, dim=0) * (2 * Nt), dim=0).real
        out["D"] = D * (tau / (2.0 * PI))
        out["D_mean"] = out["D"].mean(1)
        out["E"] = (torch.arange(2 * Nt, dtype=torch.float64, device=DEV) - Nt) * (PI / (Nt * tau))
    return out
