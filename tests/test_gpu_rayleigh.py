"""The sample solves' reported smallest eigenvalue is the Rayleigh quotient
mu = x^H G x of the vector they return, formed in double-double as the Gram is:
within half a unit in the last place of the quotient taken in exact integers.

The frames hold multiples of 2^-8, so their unit-circle evaluations come from
exact sums in any order, and the exact Gram of the solve is the one of the
evaluations that eval_unit_circle returns.  Frames of noise: the quotient is a
good part of the Gram's norm, and the double-double sums' own error (2^-100 of
that norm) is out of sight."""

from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ONE = 1 << 240


def fixed(a):
    """The entries of a (float64) times 2^240 as integers, exactly."""
    out = []
    for v in np.asarray(a, float).ravel():
        f = Fraction(float(v)) * ONE
        assert f.denominator == 1
        out.append(f.numerator)
    return out


def exact_grams(e1, e2, k1, k2):
    """G (real and imaginary parts, times 2^480) of one sample from the two frames' evaluations."""
    a = [list(zip(fixed(e.real), fixed(e.imag))) for e in (e1, e2)]

    def rho(fa, fb, l):   # sum_t conj(a_t) b_(t + l)
        x, y = a[fa], a[fb]
        re = im = 0
        for t in range(max(0, -l), min(len(x), len(y) - l)):
            p, q = x[t], y[t + l]
            re += p[0] * q[0] + p[1] * q[1]
            im += p[0] * q[1] - p[1] * q[0]
        return re, im

    N = k1 + k2
    G = [[None] * N for _ in range(N)]
    for i in range(N):
        for j in range(N):
            fa, fb = int(i >= k2), int(j >= k2)
            p, q = i - fa * k2, j - fb * k2
            if fa == fb:
                re, im = rho(fa, fa, abs(p - q))
                G[i][j] = (re, im if p >= q else -im)
            elif fa == 0:
                re, im = rho(0, 1, p - q)
                G[i][j] = (-re, -im)
            else:
                re, im = rho(0, 1, q - p)
                G[i][j] = (-re, im)
    return G


@pytest.mark.parametrize("k1,k2", [(1, 2), (4, 3), (9, 8), (13, 15)])
def test_quotient_is_correctly_rounded(k1, k2):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    m, n = 22, 18
    r = np.random.default_rng(1000 * k1 + k2)
    b1, b2 = (torch.as_tensor(r.integers(-256, 257, (m + k - 1, n + k - 1)) / 256.0, device="cuda") for k in (k1, k2))
    _, _, diag = P.recover_kernels(b1, b2, m, n, diag=True)
    S = diag["S"]
    ev = [[t.cpu().numpy() for t in P.eval_unit_circle(b, S)] for b in (b1, b2)]
    for pas in range(2):
        for j in range(0, S, 1 + S // 4):
            G = exact_grams(ev[0][pas][j], ev[1][pas][j], k1, k2)
            x = list(zip(fixed(diag["sample_vec"][pas, j].real), fixed(diag["sample_vec"][pas, j].imag)))
            mu = 0
            for i, (xr, xi) in enumerate(x):
                yr = sum(g[0] * v[0] - g[1] * v[1] for g, v in zip(G[i], x))
                yi = sum(g[0] * v[1] + g[1] * v[0] for g, v in zip(G[i], x))
                mu += xr * yr + xi * yi
            exact = Fraction(mu, ONE ** 4)
            got = Fraction(float(diag["sample_lambda0"][pas, j]))
            assert abs(got - exact) <= exact * Fraction(1, 2 ** 53), (pas, j, float((got - exact) / exact) * 2 ** 53)
