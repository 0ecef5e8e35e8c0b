"""The systematic points' division by the count n through the correctly
rounded reciprocal: q = RN(b y), r = b - q n, RN(q + r y) equals RN(b / n) for
every count the filters use (exact rational arithmetic; each float() of a
Fraction rounds correctly, as an FMA does)."""
from fractions import Fraction

import numpy as np
import pytest


def _divide(b, n):
    y = 1.0 / n
    q = b * y
    r = float(Fraction(b) - Fraction(q) * n)
    return float(Fraction(q) + Fraction(r) * Fraction(y))


@pytest.mark.parametrize("lo,hi", [(1, 64), (64, 300), (1000, 1100), (4032, 4097), (65000, 65010)])
def test_reciprocal_division_is_the_rounded_quotient(lo, hi):
    g = np.random.default_rng(lo)
    for n in range(lo, hi):
        u = g.random(6)
        total = 1.0 + g.random(6) * (n - 1)
        k = g.integers(0, n, size=6)
        bs = [float((kk + uu) * tt) for kk, uu, tt in zip(k, u, total)]
        # products next to a multiple of n and quotients next to a rounding boundary
        for q in g.random(4) * n:
            bs += [float(q * n), float(np.nextafter(q * n, 0.0)), float(np.nextafter(q * n, 1e300))]
        for b in bs:
            assert _divide(b, n) == b / n, (b, n)
