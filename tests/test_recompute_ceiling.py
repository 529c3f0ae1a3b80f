"""The stage time of the recomputing kernels as one fused multiply-add rounded towards +infinity, in exact
rational arithmetic.

For r = odd * 2^k, k <= 3, the kernels hold inv = 2^-53 * fl(fl(1 / odd) * (1 - 2^-51)) (2^-53 for odd = 1) and take
ceil(x / r) from the low bits of   y = x * inv + 2^(k - 1),   rounded up to a double.  Counts with k > 3
follow from the one with k = 3.  Values: multiples of every r and their neighbours, the top of both ranges,
and random ones."""
from fractions import Fraction

import numpy as np
import pytest


def held_reciprocal(odd: int) -> Fraction:
    return Fraction(1.0 if odd == 1 else (1.0 / odd) * (1.0 - 2.0 ** -51)) / 2 ** 53


def quotient(x: int, odd: int, k: int) -> int:
    """Mantissa field of the sum, which lies in [2^(k-1), 2^k) and is rounded up to a multiple of 2^(k-53)."""
    exact = x * held_reciprocal(odd) + Fraction(2) ** (k - 1)
    ulp = Fraction(2) ** (k - 53)
    y = -((-exact) // ulp) * ulp
    assert Fraction(2) ** (k - 1) <= y < Fraction(2) ** k
    return int((y - Fraction(2) ** (k - 1)) / ulp)


def values(top: int, r: int, g) -> list:
    xs = {0, 1, 2, r - 1, r, r + 1, top - 2, top - 1, top}
    for m in (2, 3, 1000, top // r, top // r - 1, top // (2 * r)):
        xs.update(v for v in (m * r - 1, m * r, m * r + 1) if 0 <= v <= top)
    xs.update(int(v) for v in g.integers(0, top, 300, endpoint=True))
    return sorted(xs)


@pytest.mark.parametrize("top", [(1 << 32) - 1, 1 << 40])
def test_ceiling_matches_integer_division(top):
    g = np.random.default_rng(11)
    for r in range(1, 65):
        ctz = (r & -r).bit_length() - 1
        k, odd = min(ctz, 3), r >> ctz
        for x in values(top, r, g):
            q = quotient(x, odd, k)
            rest = ctz - k
            assert (q + (1 << rest) - 1) >> rest == -(-x // r), (x, r)


def test_the_held_reciprocal_lies_just_below():
    for odd in range(3, 64, 2):
        short = 1 - held_reciprocal(odd) * 2 ** 53 * odd
        assert 0 < short < Fraction(1, 1 << 50), odd
