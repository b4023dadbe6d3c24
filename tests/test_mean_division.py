"""The kernels divide a sum S of R BF16 values by R, for R no power of two, with
Markstein's correction: q = S y (y = fp64(1/R)), then q + y (S - R q), each
step rounded once.  It equals the IEEE quotient S / R, checked here with exact
rationals on random sums and on sums one unit beside R times an FP32 midpoint."""
import random
from fractions import Fraction

import pytest


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))  # one correct rounding


@pytest.mark.parametrize("R", [3, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15])
def test_corrected_reciprocal_is_the_quotient(R):
    rng = random.Random(R)
    y = 1.0 / R

    def check(s):
        q = s * y
        assert fma(fma(-float(R), q, s), y, q) == s / R, s.hex()
    for _ in range(2000):
        check(rng.choice([-1, 1]) * float(rng.getrandbits(rng.randint(1, 53)) | 1) * 2.0 ** rng.randint(-133, 79))
        midpoint = 2 * rng.getrandbits(24) + 1
        check(float(midpoint * R + rng.choice([-1, 0, 1])) * 2.0 ** rng.randint(-133, 79))
    check(0.0)
