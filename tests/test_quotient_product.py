"""The transform's fixed-operand product (a twiddle w < q kept with its scaled
quotient wq = floor(w R / q), R = 2^(bD)).

On the CPU, a model in exact Python integers: the quotient taken from the top
columns of wq y only, the column sums below 2^64, and the limbs read from the
raw columns, at every compute limb count.  On the GPU, transforms of edge
vectors against the oracle at the limb counts where the digits fit most and
least tightly (10, 20 and 28 limbs), where the digit width changes (28, 29) and
at both ends of the limb layouts in LDS (quads, a pair, a single word)."""
import random

import pytest

import moma_inputs as mi


def shape(L, fw):
    b = 29 if L <= 28 else 28
    return b, -(-(32 * L - (0 if fw else 1)) // b)


def split(v, b, D):
    return [(v >> (b * i)) & ((1 << b) - 1) for i in range(D)]


def raw_to_limbs(raw, b, D, L, fw):
    """The kernels' limb assembly from 32-bit raw columns."""
    M = 0xFFFFFFFF
    hi = [r << (32 - b) & M for r in raw[:D - 1]]
    out = []
    for j in range(L + 1 if fw else L):
        i, s = divmod(32 * j, b)
        if i >= D:
            v = 0
        elif i == D - 1:
            v = raw[i] >> s
        else:
            have = 2 * b - s
            v = ((raw[i + 1] << 32 | hi[i]) >> (32 - b + s)) & M
            if have < 32 and i + 1 < D - 1:
                v = hi[i] >> (32 - b + s) | ((raw[i + 1] << (32 - b) & M) >> (32 - b)) << (b - s)
                v = (v | raw[i + 2] << have) & M
        out.append(v)
    return sum(v << (32 * j) for j, v in enumerate(out))


def product(y, w, q, L, fw):
    b, D = shape(L, fw)
    R, mask = 1 << (b * D), (1 << b) - 1
    a, wd, wqd, nq = split(y, b, D), split(w, b, D), split(w * R // q, b, D), split(R - q, b, D)
    m, acc = [0] * D, 0
    for c in range(D - 2, 2 * D - 1):
        acc += sum(a[j] * wqd[c - j] for j in range(max(0, c - D + 1), min(c, D - 1) + 1))
        assert acc < 2 ** 64
        if c >= D:
            m[c - D] = acc & mask
        acc >>= b
    m[D - 1] = acc
    assert acc <= mask
    raw, acc = [0] * D, 0
    for i in range(D):
        acc += sum(a[j] * wd[i - j] + m[j] * nq[i - j] for j in range(i + 1))
        assert acc < 2 ** 64
        raw[i] = acc & 0xFFFFFFFF
        acc >>= b
    raw[D - 1] &= mask
    return raw_to_limbs(raw, b, D, L, fw)


@pytest.mark.parametrize("fw", [False, True])
@pytest.mark.parametrize("L", range(1, 33))
def test_product_model_at_every_limb_count(L, fw):
    if fw and L < 2:
        pytest.skip("full-width moduli start at two limbs")
    rng = random.Random(L)
    bits = 32 * L if fw else 32 * L - 4
    for q in {(1 << bits) - 1, (1 << (bits - 1)) + 1, rng.getrandbits(bits) | 1 << (bits - 1) | 1}:
        top = q if fw else 4 * q
        pairs = [(top - 1, q - 1), (top - 1, 1), (0, q - 1), (q, q - 1)]
        pairs += [(rng.randrange(top), rng.randrange(q)) for _ in range(8)]
        for y, w in pairs:
            t = product(y, w, q, L, fw)
            assert 0 <= t < 2 * q and t % q == w * y % q


@pytest.mark.gpu
@pytest.mark.parametrize("lam", [64, 96, 160, 224, 320, 608, 640, 896, 928, 1024])
@pytest.mark.parametrize("full", [False, True])
def test_transforms_of_edge_vectors(lam, full):
    import oracle
    import paper_2501_07535_amd as moma
    from gpu_util import from_dev, say, to_dev
    f = mi.find_prime(lam, 0, bits=lam) if full else mi.find_prime(lam, 0)
    q, L, n = f.q, f.limbs, 1 << 9
    w = f.root(n)
    climbs = moma.ntt_describe(q, w, n, L)["compute_limbs"]
    rng = random.Random(lam)
    shapes = [c for c in moma.ntt_candidates(climbs, 9) if not full or (c[3] <= 2 and c[4] == 0)]
    for name, x in mi.edge_vectors(f, n, L).items():
        want = oracle.ntt_radix2(q, L, w, x)
        for s in rng.sample(shapes, 2):
            say(f"lam={lam} full={full} {name} {s}")
            moma.ntt_set_schedule(q, w, n, L, s)
            y = moma.ntt_fwd(to_dev(x), q, w)
            assert (from_dev(y) == want).all(), (name, s)
            assert (from_dev(moma.ntt_inv(y, q, w)) == x).all(), (name, s)
    moma.ntt_set_schedule(q, w, n, L, None)
