"""The shapes that small jobs take inside a batch, on both sides of each line: read
from the number of the batch's workgroups, with results against the oracle (or,
for the many, against the first job's)."""
import pytest

import moma_inputs as mi
from gpu_util import from_dev, say, to_dev

pytestmark = pytest.mark.gpu


def _batch(lam, logn, count, extra=()):
    import torch

    import paper_2501_07535_amd as moma
    f = mi.find_prime(lam, 0)
    q, L, n = f.q, f.limbs, 1 << logn
    x = mi.residues(f, n, L, 850, logn)
    d = to_dev(x)
    outs = [torch.empty_like(d) for _ in range(count)]
    jobs = [(d, o, q, f.root(n), moma.JOB_FORWARD) for o in outs]
    for ln, cnt in extra:
        e = to_dev(mi.residues(f, 1 << ln, L, 851, ln))
        jobs += [(e, torch.empty_like(e), q, f.root(1 << ln), moma.JOB_FORWARD) for _ in range(cnt)]
    b = moma.Batch(jobs)
    b.run()
    return f, x, outs, b.info()["items"]


def _items(logn, tile):
    """Workgroups of one job: one pass if its tile holds the transform, else the
    documented split of its stages with the most columns that it allows."""
    if logn <= tile:
        return 1
    for col in (5, 4, 3, 2, 1):
        passes = -(-logn // (tile - col))
        base, more = divmod(logn, passes)
        k = [base + (i < more) for i in range(passes)]
        if k[0] >= col and logn - k[0] >= col:
            return sum(1 << (logn - v - col) for v in k)


# (class, log2 points, jobs, log2 of the job's tile: 32 or 64 KiB)
CASES = [
    (256, 11, 128, 10),  # 2048 waves: two for every SIMD
    (256, 11, 129, 11),  # above: one pass in the larger tile
    (320, 10, 128, 9),   # 1024 waves
    (320, 10, 129, 10),
    (320, 16, 3, 10),    # 1536 waves, one size, a pass more in the smaller tile
    (352, 15, 8, 9),     # 2048 waves, one size, as many passes
    (1024, 10, 64, 9),   # above 16 limbs: a pass more in the smaller tile
    (1024, 12, 16, 8),   # as many
]


@pytest.mark.parametrize("lam,logn,count,tile", CASES)
def test_both_sides_of_each_line(lam, logn, count, tile):
    import oracle
    import torch
    say(f"lam={lam} logn={logn} count={count}")
    f, x, outs, items = _batch(lam, logn, count)
    assert items == count * _items(logn, tile)
    assert (from_dev(outs[0]) == oracle.ntt_radix2(f.q, f.limbs, f.root(1 << logn), x)).all()
    assert all(torch.equal(o, outs[0]) for o in outs[1:])


def test_tiny_transforms_leave_the_larger_ones_their_shape():
    """Transforms of less than a wave (64 points) beside four of 2^12 points."""
    _, _, outs, alone = _batch(256, 12, 4)
    _, _, outs2, items = _batch(256, 12, 4, extra=[(6, 5000)])
    assert items == alone + 5000
    assert (from_dev(outs2[0]) == from_dev(outs[0])).all()
