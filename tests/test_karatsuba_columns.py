"""The Karatsuba form of the transform's fixed-operand product, in exact Python
integers: of w y only the low D columns are gathered (the low halves' product
whole, the two others up to the columns that reach D), every one exact and below
2^64, and with m (R - q) added the result is the schoolbook form's."""
import random

import pytest

import moma_inputs as mi


def split(v, b, D):
    return [(v >> (b * i)) & ((1 << b) - 1) for i in range(D)]


def product(y, w, q, L):
    b = 29 if L <= 28 else 28
    D = -(-(32 * L - 1) // b)
    h, R, mask = (D + 1) // 2, 1 << (b * D), (1 << b) - 1
    g = D - h
    a, wd, wqd, nq = split(y, b, D), split(w, b, D), split(w * R // q, b, D), split(R - q, b, D)
    m, acc = [0] * D, 0
    for c in range(D - 2, 2 * D - 1):
        acc += sum(a[j] * wqd[c - j] for j in range(max(0, c - D + 1), min(c, D - 1) + 1))
        if c >= D:
            m[c - D] = acc & mask
        acc >>= b
    m[D - 1] = acc
    sa = [a[i] + (a[h + i] if i < g else 0) for i in range(h)]
    sw = [wd[i] + (wd[h + i] if i < g else 0) for i in range(h)]
    p = [0] * D
    for c in range(min(2 * h - 1, D)):
        z0 = sum(a[i] * wd[c - i] for i in range(max(0, c - h + 1), min(c, h - 1) + 1))
        p[c] += z0
        if c + h < D:
            zm = sum(sa[i] * sw[c - i] for i in range(c + 1))
            z2 = sum(a[h + i] * wd[h + c - i] for i in range(c + 1) if i < g and c - i < g)
            assert zm < 2 ** 64 and z0 + z2 <= zm
            p[c + h] += zm - z0 - z2
    for c in range(D):
        assert p[c] < 2 ** 64 and p[c] == sum(a[j] * wd[c - j] for j in range(c + 1))
    t, acc = 0, 0
    for i in range(D):
        acc += p[i] + sum(m[j] * nq[i - j] for j in range(i + 1))
        assert acc < 2 ** 64
        t, acc = t | (acc & mask) << (b * i), acc >> b
    return t


@pytest.mark.parametrize("L", range(2, 25))
def test_columns_and_result_at_every_limb_count(L):
    rng = random.Random(L)
    bits = 32 * L - 4
    for q in {mi.find_prime(32 * L, 0).q, (1 << bits) - 1, (1 << (bits - 1)) + 1}:
        pairs = [(4 * q - 1, q - 1), ((1 << (32 * L - 2)) - 1, q - 1), (0, q - 1), (q, 1)]
        pairs += [(rng.randrange(4 * q), rng.randrange(q)) for _ in range(12)]
        for y, w in pairs:
            y = min(y, 4 * q - 1)
            t = product(y, w, q, L)
            assert t < 2 * q and t % q == w * y % q
