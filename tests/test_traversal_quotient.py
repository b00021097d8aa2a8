"""Boundary times of the dense walk: the reciprocal form n y with two FMA corrections gives the rounded
quotient n / w (emulated here in exact rationals, an FMA rounding once), over the operands that the
walk admits: w of magnitude in [2^-100, 2^100) with a significand below 2 - 2^-48, n zero or of
magnitude in [2^-900, 2^900)."""
import random
from fractions import Fraction as Q

import pytest


def fma(a, b, c):
    return float(Q(a) * Q(b) + Q(c))


def quot(n, w):
    y = 1.0 / w
    q0 = n * y
    q1 = fma(fma(-w, q0, n), y, q0)
    return fma(fma(-w, q1, n), y, q1)


def _sig(rng, kind):
    """A significand in [1, 2): random, next to 1, next to 2 - 2^-48, or of few bits."""
    top = 2 ** 52 - 17
    if kind == 0:
        k = rng.randrange(top + 1)
    elif kind == 1:
        k = rng.randrange(64)
    elif kind == 2:
        k = top - rng.randrange(64)
    else:
        k = sum(1 << rng.randrange(52) for _ in range(2)) % (top + 1)
    return 1.0 + k * 2.0 ** -52


@pytest.mark.parametrize("exps", [(-3, 3), (-100, 99)])
def test_reciprocal_quotient_is_the_division(exps):
    rng = random.Random(5)
    for t in range(12000):
        w = _sig(rng, t % 4) * 2.0 ** rng.randint(*exps) * rng.choice((1, -1))
        if t % 5 == 0:     # numerators next to a product of w: quotients next to a tie or exact
            n = w * _sig(rng, (t // 4) % 4)
            n = n * (1 + rng.randint(-3, 3) * 2.0 ** -52)
        else:
            n = _sig(rng, (t // 4) % 4) * 2.0 ** rng.randint(-900 if exps[0] < -50 else -9, 899 if exps[0] < -50 else 9)
        n *= rng.choice((1, -1))
        assert quot(n, w) == n / w, (n.hex(), w.hex())
    assert quot(0.0, 1.7) == 0.0 and quot(0.0, -1.7) == 0.0
