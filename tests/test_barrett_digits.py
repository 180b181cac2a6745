"""vmul's Barrett product in digits and axpy's fixed-operand product.

On the CPU, a model in exact Python integers at every limb count: the scaling
puts the modulus on bD - 1 bits, the quotient taken from the top columns is at
most one short, every column sum stays below 2^64.  On the GPU, against the
oracle at moduli that leave 0 to 31 bits of their limbs unused (the word
scaling) and at full width, edge vectors and random ones."""
import random

import pytest

import moma_inputs as mi


def model(a, b, q, L, fw):
    bits = 29 if L <= 28 else 28
    D = -(-(32 * L - (0 if fw else 1)) // bits)
    W0 = 32 * L if fw else 32 * L - 4
    off, mask, R = bits * D - 1 - W0, (1 << bits) - 1, 1 << (bits * D)
    d = W0 - q.bit_length()
    assert 0 <= d < 32 and 0 <= off
    qn = q << (d + off)
    assert qn.bit_length() == bits * D - 1
    mu = (1 << (2 * bits * D)) // qn
    dig = lambda v, n: [(v >> (bits * i)) & mask for i in range(n)]  # noqa: E731
    mud = dig(mu, D - 1) + [mu >> (bits * (D - 1))]
    assert mud[-1] < 2 ** 31
    x, y, nq = dig(a << (d + off), D), dig(b, D), dig(R - qn, D)
    p, acc = [0] * (2 * D), 0
    for k in range(2 * D - 1):
        acc += sum(x[j] * y[k - j] for j in range(max(0, k - D + 1), min(k, D - 1) + 1))
        assert acc < 2 ** 64
        p[k], acc = acc & mask, acc >> bits
    p[-1] = acc
    assert acc <= mask
    m, acc = [0] * D, 0
    for k in range(D - 1, 2 * D):
        acc += sum(p[D - 1 + i] * mud[k - i] for i in range(k - D + 1, min(k, D) + 1))
        assert acc < 2 ** 64
        if k > D:
            m[k - D - 1] = acc & mask
        acc >>= bits
    m[D - 1] = acc
    assert acc <= mask
    t, acc = 0, 0
    for i in range(D):
        acc += p[i] + sum(m[j] * nq[i - j] for j in range(i + 1))
        assert acc < 2 ** 64
        t, acc = t | (acc & mask) << (bits * i), acc >> bits
    assert t < 2 * qn and t % (1 << off) == 0
    t >>= off
    t -= (q << d) if t >= q << d else 0
    assert t % (1 << d) == 0
    return t >> d


@pytest.mark.parametrize("fw", [False, True])
@pytest.mark.parametrize("L", range(1, 33))
def test_barrett_model_at_every_limb_count(L, fw):
    if fw and L < 2:
        pytest.skip("full-width moduli start at two limbs")
    rng = random.Random(L)
    top, low = (32 * L, 32 * L - 3) if fw else (32 * L - 4, max(2, 32 * L - 35))
    for M in {top, low, (top + low) // 2}:
        for q in {(1 << M) - 1, (1 << (M - 1)) + 1, rng.getrandbits(M) | 1 << (M - 1) | 1}:
            for a, b in [(q - 1, q - 1), (0, q - 1), (1, q - 1)] + [(rng.randrange(q), rng.randrange(q)) for _ in range(6)]:
                assert model(a, b, q, L, fw) == a * b % q


@pytest.mark.gpu
@pytest.mark.parametrize("limbs,bits", [(2, 33), (2, 59), (3, 64), (8, 229), (8, 240), (10, 316), (11, 317), (20, 636),
                                        (24, 764), (28, 892), (29, 893), (32, 997), (32, 1020),
                                        (2, 61), (7, 222), (8, 256), (21, 670), (28, 895), (29, 928), (32, 1024)])
def test_products_at_moduli_of_every_scaling(limbs, bits):
    import oracle
    import paper_2501_07535_amd as moma
    from gpu_util import from_dev, say, to_dev
    rng = random.Random(bits)
    q = rng.getrandbits(bits) | 1 << (bits - 1) | 1  # (primality plays no part in these operations)
    n = 321
    say(f"limbs={limbs} bits={bits}")
    edge = [0, 1, q - 1, q >> 1, (1 << (bits - 1)) % q, (1 << 29) % q]
    va = [rng.choice(edge) if i % 3 == 0 else rng.randrange(q) for i in range(n)]
    vb = [rng.choice(edge) if i % 5 == 0 else rng.randrange(q) for i in range(n)]
    va[:2], vb[:2] = [q - 1, q - 1], [q - 1, 1]
    a, b = mi.ints_to_rows(va, limbs), mi.ints_to_rows(vb, limbs)
    da, db = to_dev(a), to_dev(b)
    want = mi.ints_to_rows([x * y % q for x, y in zip(va, vb)], limbs)
    assert (from_dev(moma.vmul(da, db, q)) == want).all()
    outs = [to_dev(a), to_dev(a)]
    alpha = rng.randrange(q)
    batch = moma.Batch([((da, db), outs[0], q, None, moma.JOB_VMUL), ((da, db), outs[1], q, alpha, moma.JOB_AXPY)])
    batch.run()
    assert (from_dev(outs[0]) == want).all()
    for al in (alpha, 0, 1, q - 1):
        ax = mi.ints_to_rows([(al * x + y) % q for x, y in zip(va, vb)], limbs)
        assert (from_dev(moma.axpy(al, da, db, q)) == ax).all(), al
    assert (from_dev(outs[1]) == oracle.axpy(q, limbs, alpha, a, b)).all()
