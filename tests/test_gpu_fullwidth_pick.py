"""A full-width plan's initial launch shape: the best that the loaded cost model
predicts among the shapes such a modulus can run, also where the best of all is
one that it cannot (a Karatsuba form or a radix-8 unit)."""
import numpy as np
import pytest

import moma_inputs as mi
from gpu_util import from_dev, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam,logn", [(64, 14), (64, 22), (96, 13), (192, 8), (256, 8), (288, 8), (512, 12), (1024, 10)])
def test_initial_shape(lam, logn):
    import oracle
    import paper_2501_07535_amd as moma
    if not moma.load_packaged_costmodel():
        pytest.skip("no packaged cost model")
    moma.tune_db_clear()
    f = mi.find_prime(lam, 0, bits=lam)
    q, L, n = f.q, f.limbs, 1 << logn
    w = f.root(n)
    widest = 2 if L <= 16 else 1
    moma.ntt_set_schedule(q, w, n, L, None)
    got = moma.ntt_get_schedule(q, w, n, L)
    cands = []
    for s in moma.ntt_candidates(L, logn):
        if s[4] == 0 and s[3] <= widest:
            moma.ntt_set_schedule(q, w, n, L, s)  # (refused if the modulus could not run it)
            cands.append(s)
    pred = moma.costmodel_predict(np.array([moma.costmodel_features(L, logn, s) for s in cands], np.float32))
    say(f"full width {lam} bits 2^{logn}: {got}")
    moma.ntt_set_schedule(q, w, n, L, None)
    assert got == moma.ntt_get_schedule(q, w, n, L) == cands[int(np.argmin(pred))]
    if logn <= 14:
        x = mi.residues(f, n, L, 860, logn)
        assert (from_dev(moma.ntt_fwd(to_dev(x), q, w)) == oracle.ntt_radix2(q, L, w, x)).all()
