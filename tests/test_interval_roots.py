"""pm_chernoff_interval (host) against its defining equation k D(count / k, p)
= ln(1 / delta), solved in 60-digit arithmetic: roots near and far from the
observed proportion, on both sides of the switch between the two iterations.

Tolerance: the observed proportion and the target are rounded once each
(relative 2^-53), and the root moves by at most 1 + target / alpha times that
(the lower root; target / beta for one minus the upper root), so 16 roundings
of that size are allowed."""
from decimal import Decimal, getcontext

import pytest

from paper_1411_4942_amd import pathsamp as ps

ONE = Decimal(1)


def _roots(count, k, delta):
    getcontext().prec = 60
    t = -Decimal(delta).ln() / k
    a = Decimal(count) / k

    def far(a):  # the root p < a
        x0, x1 = Decimal(-3000), Decimal(0)  # p = a e^x
        for _ in range(180):
            x = (x0 + x1) / 2
            p = a * x.exp()
            if a * -x + (1 - a) * ((1 - a) / (1 - p)).ln() > t:
                x0 = x
            else:
                x1 = x
        return p

    return far(a), far(1 - a)  # p_lo, 1 - p_hi


@pytest.mark.parametrize("delta", [0.01, 0.5, 1e-12, 0.999])
@pytest.mark.parametrize("count,k", [(1, 2), (1, 3), (1, 7), (1, 1000), (2, 1000), (5, 1000), (18, 1000), (37, 1000),
                                     (500, 1000), (963, 1000), (999, 1000), (200, 200000), (66666, 200000),
                                     (199999, 200000), (1, 10**7), (40, 10**7), (3 * 10**6, 10**7), (10**9, 10**18)])
def test_roots_solve_the_equation(count, k, delta):
    lo, hi = ps.chernoff_interval(count, k, delta)
    p, q = _roots(count, k, delta)
    t = float(-Decimal(delta).ln() / k)
    alpha, beta = count / k, (k - count) / k
    eps = 2.0 ** -53
    assert lo < alpha < hi
    assert abs(float((Decimal(lo) - p) / p)) <= 16 * eps * (1 + t / alpha)
    upper = ONE - q
    assert abs(float((Decimal(hi) - upper) / upper)) <= 16 * eps * (1 + t / beta)


def test_ends():
    for k in (1, 10, 12345):
        assert ps.chernoff_interval(0, k, 0.01)[0] == 0.0
        assert ps.chernoff_interval(k, k, 0.01)[1] == 1.0
    # targets beyond every double of (0, 1): the ends themselves
    assert ps.chernoff_interval(1, 2, 1e-300)[1] == 1.0
