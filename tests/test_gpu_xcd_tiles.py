"""GPU parity around the rule that keeps the tiles sharing a line on one XCD: as
many groups of tiles as the rule needs, half as many and more, for each number
of columns, in a lone call, in place and in a batch."""
import pytest

import moma_inputs as mi
from gpu_util import from_dev, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("logn", [9, 11, 13, 14])
def test_tiles_cover_the_transform(cols, logn):
    import oracle
    import paper_2501_07535_amd as moma
    f = mi.find_prime(128, 0)
    q, L, n = f.q, f.limbs, 1 << logn
    w = f.root(n)
    shapes = [c for c in moma.ntt_candidates(L, logn) if c[1] == cols and c[0] < logn and c[4] == 0 and c[3] == 1]
    if not shapes:
        pytest.skip("no multi-pass shape with these columns")
    x = mi.residues(f, n, L, 810, logn)
    want = oracle.ntt_radix2(q, L, w, x)
    for s in (shapes[0], shapes[-1]):
        say(f"logn={logn} {s}")
        moma.ntt_set_schedule(q, w, n, L, s)
        d = to_dev(x)
        assert (from_dev(moma.ntt_fwd(d, q, w)) == want).all(), s
        assert (from_dev(moma.ntt_fwd(d, q, w, out=d)) == want).all(), s
    moma.ntt_set_schedule(q, w, n, L, None)
    ins = [to_dev(x) for _ in range(3)]
    outs = [to_dev(x) for _ in range(3)]
    b = moma.Batch([(i, o, q, w, moma.JOB_FORWARD) for i, o in zip(ins, outs)])
    b.run()
    assert all((from_dev(o) == want).all() for o in outs)
