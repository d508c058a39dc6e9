"""The direction table's quotient (a correctly rounded reciprocal, one
product and one fused correction) against division, in exact arithmetic."""
import math
import random
from fractions import Fraction as F

import pytest


def _quot(n, d):
    """dir_quot's operations, each rounded to double (float(Fraction) rounds to nearest even)."""
    r = 1.0 / d
    q = n * r
    rem = float(F(n) - F(q) * F(d))
    return float(F(rem) * F(r) + F(q))


@pytest.mark.parametrize("lo,hi", [(-20, 5), (-50, -20), (-3, 1)])
def test_quotient_is_the_division(lo, hi):
    """Operands as the walks meet them: positions and offsets up to tens of
    mm (down to the rounding of cancelled ones), direction components."""
    rng = random.Random(lo)
    for k in range(20000):
        n = math.ldexp(rng.random() + 0.5, rng.randint(lo, hi)) * rng.choice((-1, 1))
        d = math.ldexp(rng.random() + 0.5, rng.choice((0, 0, 0, -1, -3, -10, -40))) * rng.choice((-1, 1))
        if k % 4 == 0:           # near-ties and small integers
            n, d = float(rng.randint(1, 1 << 24)), float(rng.randint(1, 1 << 10))
        if k % 16 == 1:          # mantissas next to a power of two
            d = math.nextafter(math.ldexp(1.0, rng.randint(-4, 0)), rng.choice((0.0, 2.0)))
        assert _quot(n, d) == n / d, (n, d)
