"""GPU parity of passes with two columns per tile, whose lines 16 neighbouring
tiles share: the widest group that is kept on one XCD (set_schedule and the
batches take such shapes, the tuner's list does not), with fewer tiles than 8
groups need, just as many, and more."""
import pytest

import moma_inputs as mi
from gpu_util import from_dev, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam,full", [(64, False), (128, False), (256, True), (1024, False)])
@pytest.mark.parametrize("logn,tile", [(7, 5), (10, 6), (11, 6), (12, 7), (13, 6)])
def test_two_columns(lam, full, logn, tile):
    import oracle
    import paper_2501_07535_amd as moma
    f = mi.find_prime(lam, 0, bits=lam) if full else mi.find_prime(lam, 0)
    q, L, n = f.q, f.limbs, 1 << logn
    w = f.root(n)
    x = mi.residues(f, n, L, 840, logn)
    want = oracle.ntt_radix2(q, L, w, x)
    for threads in (64, 128):
        s = (tile, 1, threads, 1, 0)
        say(f"lam={lam} full={full} logn={logn} {s}")
        moma.ntt_set_schedule(q, w, n, L, s)
        d = to_dev(x)
        y = moma.ntt_fwd(d, q, w)
        assert (from_dev(y) == want).all(), s
        assert (from_dev(moma.ntt_inv(y, q, w)) == x).all(), s
        moma.ntt_fwd(d, q, w, out=d)
        assert (from_dev(d) == want).all(), s
    moma.ntt_set_schedule(q, w, n, L, None)
