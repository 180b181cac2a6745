"""The work a user of this library has it do, as timed cases.

Every case is a call (or a short chain of calls) of the public Python entry
points on data that is already on the GPU: single transforms from the smallest
to the largest sizes, both directions, narrow to wide moduli, full-width moduli,
the cyclic product, a mixed batch, elementwise operations, and the conversion
of element-major integers around them.

A case is a dict of plain values:
  kind    "fwd", "inv" (transforms), "mul" (cyclic product), "blas",
          "elements" (pack, operate, unpack) or "batch"
  bits    the width class; q has bits - 4 bits, or exactly `bits` where
          "full" is set; residues are stored in bits / 32 words
  logn    log2 of a transform's points; n: an elementwise call's elements
  op      the elementwise operation
  jobs    a batch's number of jobs; shape: where its sequence of shapes starts
"""
import functools
import math
import random

import numpy as np
import torch

import paper_2501_07535_amd as moma

BATCH_BITS = (64, 128, 256, 384)  # the mixed batch's width classes and sizes
BATCH_LOGN = tuple(range(10, 17))
OPS = ("vadd", "vsub", "vmul", "axpy")


def listed():
    return [
        # one short transform, as a program that needs a single product or
        # evaluation now issues it: launches and latency
        {"name": "fwd256_2e12", "kind": "fwd", "bits": 256, "full": False, "logn": 12},
        {"name": "inv384_2e14", "kind": "inv", "bits": 384, "full": False, "logn": 14},
        # the middle of the range, too small to fill the chip by itself
        {"name": "fwd256_2e16", "kind": "fwd", "bits": 256, "full": False, "logn": 16},
        # the size a proof system or the benchmark transforms
        {"name": "fwd256_2e20", "kind": "fwd", "bits": 256, "full": False, "logn": 20},
        # narrow residues, a long transform: closest to memory
        {"name": "inv128_2e22", "kind": "inv", "bits": 128, "full": False, "logn": 22},
        # the largest transform of the 256-bit sweep
        {"name": "fwd256_2e24", "kind": "fwd", "bits": 256, "full": False, "logn": 24},
        # the widest residues: arithmetic and registers
        {"name": "fwd1024_2e20", "kind": "fwd", "bits": 1024, "full": False, "logn": 20},
        # a modulus that uses every bit of its storage
        {"name": "inv256full_2e20", "kind": "inv", "bits": 256, "full": True, "logn": 20},
        # polynomial multiplication with wide coefficients
        {"name": "mul768_2e16", "kind": "mul", "bits": 768, "full": False, "logn": 16},
        # many independent transforms of mixed widths and sizes in one graph
        {"name": "batch256", "kind": "batch", "jobs": 256, "shape": 0},
        # elementwise products over long vectors
        {"name": "vmul768_2e24", "kind": "blas", "bits": 768, "full": False, "n": 1 << 24, "op": "vmul"},
        # data held as an array of integers: converted, used once, converted back
        {"name": "elements256_1000003", "kind": "elements", "bits": 256, "full": False, "n": 1000003, "op": "axpy"},
    ]


def _weight(c):
    """A case's cost relative to others: butterflies or products times their words."""
    words = c["bits"] // 32
    if c["kind"] in ("blas", "elements"):
        return c["n"] * (words * words + 12 * words) * (2 if c["kind"] == "elements" else 1)
    return (c["logn"] << c["logn"]) * (words * words + 12 * words) // 2 * (3 if c["kind"] == "mul" else 1)


def draw(rng):
    kind = rng.choice(("fwd", "fwd", "inv", "inv", "mul", "blas", "blas", "elements", "batch"))
    if kind == "batch":
        return {"kind": kind, "jobs": round(2 ** rng.uniform(1, 8)), "shape": rng.randrange(1, 1 << 20)}
    c = {"kind": kind, "bits": 32 * rng.randint(2, 32), "full": rng.random() < 0.2}
    if kind in ("blas", "elements"):
        c["n"] = round(2 ** rng.uniform(8, 24))
        c["op"] = rng.choice(OPS)
    else:
        c["logn"] = rng.randint(8, 24)
    # no larger than half of the largest listed transform or elementwise call
    cap = _weight({"kind": "fwd", "bits": 256, "logn": 24}) // 2
    while _weight(c) > cap:
        if "n" in c:
            c["n"] = c["n"] * 3 // 4
        else:
            c["logn"] -= 1
    return c


# ------------------------------------------------------------------ moduli

def _is_prime(n, rng):
    if any(n % p == 0 for p in (3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37, 41, 43, 47)):
        return n in (3, 5, 7, 11, 13)
    d, s = n - 1, 0
    while d % 2 == 0:
        d, s = d // 2, s + 1
    for _ in range(20):
        x = pow(rng.randrange(2, n - 1), d, n)
        if x in (1, n - 1):
            continue
        for _ in range(s - 1):
            x = x * x % n
            if x == n - 1:
                break
        else:
            return False
    return True


@functools.lru_cache(maxsize=None)
def _modulus(bits, full, index=0):
    """A prime q = c 2^32 + 1 of the class and a quadratic non-residue."""
    m = bits if full else bits - 4
    rng = random.Random(1000 * m + index)
    c = (1 << (m - 33)) + rng.randrange(1 << (m - 33))
    while not _is_prime((c << 32) + 1, rng):
        c += 1
    q = (c << 32) + 1
    assert q.bit_length() == m
    z = 2
    while pow(z, (q - 1) // 2, q) != q - 1:
        z += 1
    return q, z


@functools.lru_cache(maxsize=None)
def _root(bits, full, index, n):
    q, z = _modulus(bits, full, index)
    return pow(z, (q - 1) // n, q)


def _batch_shapes(case):
    """(bits, log2 n, prime index, inverse) of each job."""
    rng = random.Random(20250107 + case["shape"])
    return [(rng.choice(BATCH_BITS), rng.choice(BATCH_LOGN), rng.randrange(2), rng.random() < 0.25)
            for _ in range(case["jobs"])]


# ------------------------------------------------------------------ inputs

def _residues(gen, q, limbs, n):
    """n uniform residues below q's top word, (limbs, n) words."""
    x = torch.randint(-(1 << 31), 1 << 31, (limbs, n), dtype=torch.int32, device="cuda", generator=gen)
    top = q >> (32 * (limbs - 1))
    hi = torch.randint(0, top, (n,), dtype=torch.int64, device="cuda", generator=gen)
    x[limbs - 1] = torch.where(hi >= 1 << 31, hi - (1 << 32), hi).to(torch.int32)
    return x


def _alpha(seed, q):
    return random.Random(seed).randrange(q)


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _inputs(case, seed):
    """The case's input vectors, limb-planar (element-major for "elements")."""
    gen = _gen(seed)
    if case["kind"] == "batch":
        return [_residues(gen, _modulus(b, False, i)[0], b // 32, 1 << ln) for b, ln, i, _ in _batch_shapes(case)]
    q, limbs = _modulus(case["bits"], case["full"])[0], case["bits"] // 32
    n = case["n"] if "n" in case else 1 << case["logn"]
    xs = [_residues(gen, q, limbs, n) for _ in range(1 if case["kind"] in ("fwd", "inv") else 2)]
    if case["kind"] == "elements":
        xs = [x.t().contiguous() for x in xs]
    return xs


def prepare(case, seed):
    xs = _inputs(case, seed)
    st = {"kind": case["kind"], "xs": xs}
    if case["kind"] == "batch":
        # the jobs' outputs side by side in one buffer, as a program would send them on
        st["out"] = torch.empty(sum(x.numel() for x in xs), dtype=torch.int32, device="cuda")
        outs = [y.view_as(x) for x, y in zip(xs, st["out"].split([x.numel() for x in xs]))]
        st["batch"] = moma.Batch([(x, y, _modulus(b, False, i)[0], _root(b, False, i, 1 << ln),
                                   moma.JOB_INVERSE if inv else moma.JOB_FORWARD)
                                  for x, y, (b, ln, i, inv) in zip(xs, outs, _batch_shapes(case))])
        return st
    q, limbs = _modulus(case["bits"], case["full"])[0], case["bits"] // 32
    st["q"] = q
    st["out"] = torch.empty_like(xs[0])
    if "logn" in case:
        st["w"] = _root(case["bits"], case["full"], 0, 1 << case["logn"])
        moma.ntt_prepare(q, st["w"], 1 << case["logn"], limbs)
    else:
        st["op"] = case["op"]
        st["alpha"] = _alpha(seed, q)
        if case["kind"] == "elements":
            st["planar"] = [torch.empty((limbs, case["n"]), dtype=torch.int32, device="cuda") for _ in range(3)]
    return st


def _elementwise(st, a, b, out):
    if st["op"] == "axpy":
        return moma.axpy(st["alpha"], a, b, st["q"], out=out)
    return getattr(moma, st["op"])(a, b, st["q"], out=out)


def run(st):
    kind, xs = st["kind"], st["xs"]
    if kind == "fwd":
        return moma.ntt_fwd(xs[0], st["q"], st["w"], out=st["out"])
    if kind == "inv":
        return moma.ntt_inv(xs[0], st["q"], st["w"], out=st["out"])
    if kind == "mul":
        return moma.ntt_cyclic_mul(xs[0], xs[1], st["q"], st["w"], out=st["out"])
    if kind == "batch":
        st["batch"].run()
        return st["out"]
    if kind == "elements":
        a, b, c = st["planar"]
        moma.pack(xs[0], out=a)
        moma.pack(xs[1], out=b)
        return moma.unpack(_elementwise(st, a, b, c), out=st["out"])
    return _elementwise(st, xs[0], xs[1], st["out"])


# ------------------------------------------------------------------ accounts

def _transform_work(words, logn):
    """One transform: data read and written once; a butterfly is a modular
    multiply (2 words^2 + words word products, two operations each), an
    addition and a subtraction (3 words operations each)."""
    n = 1 << logn
    return 8 * words * n, n // 2 * logn * (2 * (2 * words * words + words) + 6 * words)


def work(case):
    if case["kind"] == "batch":
        parts = [_transform_work(b // 32, ln) for b, ln, _, _ in _batch_shapes(case)]
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    words = case["bits"] // 32
    if "logn" in case:
        nbytes, flops = _transform_work(words, case["logn"])
        if case["kind"] == "mul":
            n = 1 << case["logn"]
            return {"bytes": 12 * words * n, "flops": 3 * flops + n * 2 * (2 * words * words + words)}
        return {"bytes": nbytes, "flops": flops}
    per = 3 * words + (2 * (2 * words * words + words) if case["op"] in ("vmul", "axpy") else 0)
    return {"bytes": 12 * words * case["n"], "flops": per * case["n"]}


def _ints(x):
    """(limbs, n) words as an object array of Python integers."""
    raw = np.ascontiguousarray(x.cpu().numpy().T).tobytes()
    size = 4 * x.shape[0]
    out = np.empty(x.shape[1], dtype=object)
    for i in range(x.shape[1]):
        out[i] = int.from_bytes(raw[i * size:(i + 1) * size], "little")
    return out


def _planar(v, limbs):
    raw = b"".join(int(e).to_bytes(4 * limbs, "little") for e in v)
    return torch.from_numpy(np.frombuffer(raw, dtype="<i4").reshape(-1, limbs).T.copy())


def _transform(v, q, w):
    """sum_j v[j] w^(jk) for every k, by halving the output index's parity."""
    n = len(v)
    pw = np.ones(max(1, n // 2), dtype=object)
    step = 1
    while step < n // 2:  # powers of w, doubling
        pw[step:2 * step] = pw[:step] * pow(w, step, q) % q
        step *= 2
    x, size = v.reshape(1, n), n
    while size > 1:
        h = size // 2
        a, b = x[:, :h], x[:, h:]
        x = np.concatenate([(a + b) % q, (a - b) * pw[::n // size][:h] % q])
        size = h
    return x.reshape(n)  # row r holds k with its low bits in r: already in order


def exact(case, seed):
    if case["kind"] == "batch" or work(case)["flops"] > 1.2e9:
        return None  # too long in Python integers
    q, limbs = _modulus(case["bits"], case["full"])[0], case["bits"] // 32
    xs = _inputs(case, seed)
    if case["kind"] == "elements":
        xs = [x.t() for x in xs]
    v = [_ints(x) for x in xs]
    if "logn" in case:
        n = 1 << case["logn"]
        w = _root(case["bits"], case["full"], 0, n)
        if case["kind"] == "fwd":
            r = _transform(v[0], q, w)
        else:
            y = v[0] if case["kind"] == "inv" else _transform(v[0], q, w) * _transform(v[1], q, w) % q
            r = _transform(y, q, pow(w, -1, q)) * pow(n, -1, q) % q
    else:
        a, b = v
        r = {"vadd": lambda: a + b, "vsub": lambda: a - b, "vmul": lambda: a * b,
             "axpy": lambda: _alpha(seed, q) * a + b}[case["op"]]() % q
    out = _planar(r, limbs)
    return out.t().contiguous() if case["kind"] == "elements" else out
