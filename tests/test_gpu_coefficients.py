"""GPU: Chebyshev coefficients far past the truncation, down to the smallest
normal numbers.  (-i)^n 2 J_n(x) by downward recurrence carries a rounding per
order and the growth of none (the recurrence is stable downwards): 4 (n + 8)
roundings of 2^-53 relative, against the power series

  J_n(x) = (x/2)^n / n! sum_m (-x^2/4)^m / (m! (n+1)..(n+m)),  n > x,

in exact rationals down to terms of 2^-200 (the sum is above 2^-50)."""
from fractions import Fraction

import numpy as np
import pytest

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


def bessel(n, x):
    h = Fraction(x) / 2
    term, total, m = Fraction(1), Fraction(0), 0
    while abs(term) > Fraction(1, 1 << 200):
        total += term
        m += 1
        term *= -h * h / (m * (n + m))
    f = total * h ** n
    for k in range(2, n + 1):
        f /= k
    return f


@pytest.mark.parametrize("x,nmax", [(np.pi, 200), (1.0, 150), (10.0, 300), (0.01, 90),
                                    (100.0, 600), (1e-3, 60)])
def test_coefficients_past_the_truncation(csp, ctx, x, nmax):
    print("[gpu] coefficients x=%g nmax=%d" % (x, nmax), flush=True)
    c, _ = csp.csp_chebyshev_coefficients(ctx, x, nmax)
    c = c.cpu().numpy()
    for n in range(int(x) + 1, nmax + 1, 7):
        ref = 2 * bessel(n, x)
        if ref < Fraction(1, 2 ** 1021):
            break
        got = c[n] * (1, 1j, -1, -1j)[n % 4]
        assert got.imag == 0.0
        assert abs(Fraction(float(got.real)) / ref - 1) < Fraction(4 * (n + 8), 1 << 53), n
