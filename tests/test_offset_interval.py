"""The bounds that the offset form's comments state, in exact Python integers, at
the operands where they are tightest: the quotient estimate falls one short for x
up to 19 2^-27 above a multiple of q (1.19e-7 of q, for a q just above a power of
two), and the product's dropped columns weigh up to (D - 2) 2^-b of q.  What the
kernels rely on is less tight: 1/64 for each."""
from fractions import Fraction

import pytest


def shape(L):
    b = 29 if L <= 28 else 28
    return b, -(-(32 * L - 1) // b)


LIMBS = [L for L in range(6, 33) if shape(L)[0] * shape(L)[1] >= 32 * L]


@pytest.mark.parametrize("L", LIMBS)
def test_estimate_at_the_end_of_its_interval(L):
    M = 32 * L - 4
    worst = Fraction(0)
    for q in ((1 << (M - 1)) + 1, (1 << (M - 1)) + (1 << (M - 28)) - 1, (1 << M) - 1, 3 << (M - 2) | 1):
        cinv = (1 << 58) // ((q >> (32 * (L - 1))) + 1)
        def estimate(x):
            return ((x >> (32 * (L - 1))) * cinv >> 32) >> 26
        for k in range(16):
            # the largest excess e with floor((k q + e) / q) - 1 still returned
            lo, hi = -1, q
            while hi - lo > 1:
                mid = (lo + hi) // 2
                lo, hi = (mid, hi) if estimate(k * q + mid) < k else (lo, mid)
            assert estimate(k * q + hi) == k  # one short below hi, exact from there on
            worst = max(worst, Fraction(hi, q))
            for x in (k * q, k * q + hi - 1, k * q + hi, k * q + q - 1):
                assert 0 <= x // q - estimate(x) <= (1 if x % q < hi else 0)
    assert worst < Fraction(19, 1 << 27)
    assert worst > Fraction(1, 1 << 24)  # (2^-24 would be too tight a bound)
    assert worst < Fraction(1, 64)


@pytest.mark.parametrize("L", LIMBS)
def test_product_slack(L):
    b, D = shape(L)
    # columns 0 .. D-3 of the quotient's product, all digits largest, in units of R
    low = sum((c + 1) * ((1 << b) - 1) ** 2 << (b * c) for c in range(D - 2))
    slack = Fraction(low, 1 << (b * D))
    assert slack < Fraction(D - 2, 1 << b) < Fraction(1, 64)
