"""1 / n of the region counts: one Newton step in float32 from any start within one
ulp of 1 / n gives the correctly rounded reciprocal, for every count a region can
have.  Exact rational arithmetic, CPU only."""
from fractions import Fraction

import numpy as np

L_MAX = 17


def rn(x):
    """x (a Fraction) rounded to float32, nearest even."""
    y = np.float32(float(x))
    near = (np.nextafter(y, np.float32(-np.inf)), y, np.nextafter(y, np.float32(np.inf)))
    return min(near, key=lambda c: (abs(Fraction(float(c)) - x), int(c.view(np.uint32)) & 1))


def test_newton_step_rounds_correctly():
    for n in range(1, (2 * L_MAX + 1) ** 2 + 1):
        want = rn(Fraction(1, n))
        for y in (np.nextafter(want, np.float32(0)), want, np.nextafter(want, np.float32(2))):
            y = Fraction(float(y))
            e = Fraction(float(rn(1 - n * y)))
            assert rn(e * y + y) == want, n
