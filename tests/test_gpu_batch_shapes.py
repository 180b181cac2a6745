"""GPU parity of batches on both sides of the line where a limb count's jobs
take the sparse launch shapes (waves of radix-2 units below four per SIMD), at
the limb counts on both sides of the radix-4 rule and at full width."""
import pytest

import moma_inputs as mi
from gpu_util import from_dev, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam,full", [(64, False), (256, False), (288, False), (384, False), (512, False), (1024, False),
                                      (256, True)])
@pytest.mark.parametrize("dense", [False, True])
def test_batches_around_the_sparse_line(lam, full, dense):
    import oracle
    import paper_2501_07535_amd as moma
    f = mi.find_prime(lam, 0, bits=lam) if full else mi.find_prime(lam, 0)
    q, L = f.q, f.limbs
    sizes = [2, 1 << 8, 1 << 10, 1 << 11]
    # the waves that cross the line come from large jobs that are checked by their round trip
    big, count = 1 << 16, 9 if dense else 0
    say(f"lam={lam} full={full} dense={dense}")
    jobs, checks = [], []
    for n in sizes:
        x = mi.residues(f, n, L, 830, n)
        d, o = to_dev(x), to_dev(x)
        jobs.append((d, o, q, f.root(n), moma.JOB_FORWARD))
        checks.append((o, oracle.ntt_radix2(q, L, f.root(n), x)))
        i = to_dev(x)
        jobs.append((i, i, q, f.root(n), moma.JOB_INVERSE))
        checks.append((i, oracle.intt_radix2(q, L, f.root(n), x)))
        p = to_dev(x)
        jobs.append(((d, d), p, q, f.root(n), moma.JOB_CYCLIC_MUL))
        y = oracle.ntt_radix2(q, L, f.root(n), x)
        checks.append((p, oracle.intt_radix2(q, L, f.root(n), oracle.vmul(q, L, y, y))))
    w = f.root(big)
    xb = mi.residues(f, big, L, 831, 0)
    db = to_dev(xb)
    outs = [to_dev(xb) for _ in range(count)]
    jobs += [(db, o, q, w, moma.JOB_FORWARD) for o in outs]
    b = moma.Batch(jobs)
    b.run()
    for k, (o, want) in enumerate(checks):
        assert (from_dev(o) == want).all(), k
    for o in outs:
        assert (from_dev(moma.ntt_inv(o, q, w)) == xb).all()
