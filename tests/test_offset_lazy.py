"""The offset form of the lazy butterflies (values in [0, 16q)).

On the CPU, in exact Python integers: the reduction's estimate and result, the
product's bound for operands up to 16q, and the bounds over every sequence of
rounds a pass can run.  On the GPU, edge vectors against the oracle at the limb
counts on both sides of the rule, in passes short and long enough to reduce
once, twice and more, lone, in a cyclic product and in a batch."""
import random

import pytest

import moma_inputs as mi


def spare(L):
    b = 29 if L <= 28 else 28
    return b * -(-(32 * L - 1) // b) - 32 * L


def growth(L):
    return 64 + (64 >> min(6, spare(L))) + 1


LIMBS = [L for L in range(1, 33) if spare(L) >= 0]


@pytest.mark.parametrize("L", LIMBS)
def test_reduction_and_product_bounds(L):
    rng = random.Random(L)
    b, R = 29 if L <= 28 else 28, 1 << (32 * L + spare(L))
    D = (32 * L + spare(L)) // b
    for M in {32 * L - 4, max(2, 32 * L - 35), 32 * L - 20}:
        for q in {(1 << M) - 1, (1 << (M - 1)) + 1, rng.getrandbits(M) | 1 << (M - 1) | 1}:
            d = 32 * L - 4 - M
            qt = (q << d) >> (32 * (L - 1))
            assert 2 ** 27 <= qt < 2 ** 28
            cinv = (1 << 58) // (qt + 1)
            assert cinv < 2 ** 32
            words, carry = [], 0
            for i in range(L):
                v = (q >> (32 * i) & 0xFFFFFFFF) + carry
                words.append((v & 0xFFFFFFFF) - ((v >> 31 & 1) << 32))
                carry = 1 if v >> 31 else 0
            assert carry == 0 and sum(w << (32 * i) for i, w in enumerate(words)) == q
            edges = [k * q + e for k in range(16) for e in (0, 1, q - 1)]
            for x in edges + [rng.randrange(16 * q) for _ in range(20)]:
                xt = (x << d) >> (32 * (L - 1))
                assert xt < 2 ** 32
                f = (xt * cinv >> 32) >> 26
                for off in (0, 7):
                    r, acc = 0, 0
                    for i in range(L):
                        acc = (acc >> 32) + (off - f) * words[i]
                        assert -2 ** 63 <= acc < 2 ** 63
                        r += (acc & 0xFFFFFFFF) << (32 * i)
                    r = (x + r) % (1 << (32 * L))
                    assert r % q == x % q and 64 * r <= (64 * (off + 1) + 1) * q and r >= off * q
                    assert off or r < 2 * q
            # the product of y < 16q, its quotient cut to the columns from D - 2
            for w in (q - 1, q // 2, rng.randrange(1, q)):
                wq = w * R // q
                for y in (16 * q - 1, 15 * q + 1, rng.randrange(16 * q)):
                    low = sum(((y >> b * i) & (2 ** b - 1)) * ((wq >> b * j) & (2 ** b - 1)) << (b * (i + j))
                              for i in range(D) for j in range(D) if i + j < D - 2)
                    t = w * y - (wq * y - low) // R * q
                    assert 0 <= t and 64 * t < growth(L) * q and t < 2 * q


@pytest.mark.parametrize("L", LIMBS)
@pytest.mark.parametrize("first", [False, True])
def test_bounds_over_every_sequence_of_rounds(L, first):
    g = growth(L)

    def walk(left, lo, hi, start):
        if left == 0:
            return
        for r in (1, 2, 3):
            if r > left:
                continue
            if start and first:
                walk(left - r, 0, 128 * r, False)
                continue
            a, b = lo, hi
            if a < r * g or b + r * g > 1024:
                a, b = 448, 513
            a, b = a - r * g, b + r * g
            assert a >= 0 and b <= 1024
            walk(left - r, a, b, False)

    walk(13, 0, 1024, True)


@pytest.mark.gpu
@pytest.mark.parametrize("lam,logn", [(160, 11), (192, 11), (256, 12), (288, 11), (320, 10), (608, 10), (640, 10), (896, 10),
                                      (928, 9), (1024, 11)])
def test_edge_vectors_at_both_sides_of_the_rule(lam, logn):
    import oracle
    import paper_2501_07535_amd as moma
    from gpu_util import from_dev, say, to_dev
    f = mi.find_prime(lam, 0)
    q, L, n = f.q, f.limbs, 1 << logn
    w = f.root(n)
    cands = [c for c in moma.ntt_candidates(L, logn) if c[4] == 0 and c[3] <= 2]
    rng = random.Random(lam)
    one = [c for c in cands if c[0] >= logn]
    shapes = ([max(one)] if one else []) + rng.sample([c for c in cands if c[0] < logn], 3)
    vecs = mi.edge_vectors(f, n, L)
    vecs["random"] = mi.residues(f, n, L, 820, 0)
    for name in ("all_qm1", "alt_0_qm1", "carry_run", "random"):
        x = vecs[name]
        want = oracle.ntt_radix2(q, L, w, x)
        sq = oracle.intt_radix2(q, L, w, oracle.vmul(q, L, want, want))
        for s in shapes:
            say(f"lam={lam} {name} {s}")
            moma.ntt_set_schedule(q, w, n, L, s)
            d = to_dev(x)
            y = moma.ntt_fwd(d, q, w)
            assert (from_dev(y) == want).all(), (name, s)
            assert (from_dev(moma.ntt_inv(y, q, w)) == x).all(), (name, s)
            assert (from_dev(moma.ntt_cyclic_mul(d, d, q, w)) == sq).all(), (name, s)
        moma.ntt_set_schedule(q, w, n, L, None)
        d, o = to_dev(x), to_dev(x)
        b = moma.Batch([(d, o, q, w, moma.JOB_FORWARD)])
        b.run()
        assert (from_dev(o) == want).all(), name
