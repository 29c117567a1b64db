"""Parton fractions of the inverse CDF against an extended-precision solution of F(x) - F(tau) = u Z for
each draw, over exponents from those of a flat density (no factor of 1 - x) to steep ones."""
from math import comb

import numpy as np
import pytest

from oracle import draws, pdf

pytestmark = pytest.mark.gpu
LD = np.longdouble


def solve(u, tau, a, b):
    """x and the size of the primitive's terms over x f(x), in long double."""
    a, tau, u = LD(a), LD(tau), u.astype(LD)
    coef = [LD((-1) ** k * comb(b, k)) / (a + k + 1) for k in range(b + 1)]

    def F(x):
        p = coef[-1]
        for c in coef[-2::-1]:
            p = p * x + c
        return x ** (a + 1) * p

    F1, Ft = F(LD(1)), F(tau)
    Z = F1 - Ft
    lo, hi = np.full(u.shape, np.log(tau)), np.zeros(u.shape, LD)
    for _ in range(70):
        y = (lo + hi) / 2
        g = F(np.exp(y)) - Ft - u * Z
        lo, hi = np.where(g < 0, y, lo), np.where(g < 0, hi, y)
    x = np.exp((lo + hi) / 2)
    f = x ** a * (1 - x) ** b
    return x, (max(abs(F1), abs(Ft)) + abs(F(x))) / (x * f)


@pytest.mark.parametrize("n,a,b", [(4, -1.3, 5), (8, -1.3, 5), (12, -1.3, 5), (5, -0.5, 3), (6, 0.3, 2), (7, -1.7, 8),
                                   (4, 0.0, 0)])
def test_fractions(gpu_lib, n, a, b):
    N = (1 << 14) + 77
    c = gpu_lib.config(n, seed=77, pdf_a=a, pdf_b=b)
    print("density", n, a, b, flush=True)
    x = gpu_lib.generate(c, N, outputs=("x12",))["x12"].cpu().numpy()
    u = draws.split_draws(draws.event_words(77, np.arange(N), n), n)[0]
    ref, cond = solve(u, pdf.tau_min(n, 20.0, 14000.0), a, b)
    err = np.abs((x - ref) / ref).astype(np.float64)
    # 2^-53 per rounding: a few of x itself, and of the primitive's terms as the equation passes them on
    bound = 2.0 ** -53 * (8.0 + 16.0 * cond.astype(np.float64))
    print(f"max error {err.max():.2e}, rms {np.sqrt((err ** 2).mean()):.2e}, of its bound {(err / bound).max():.3f}")
    assert (err <= bound).all()
    assert (x > 0).all() and (x < 1).all()
