"""A full-width plan's initial launch shape: the loaded cost model's pick, without
the Karatsuba form that such a modulus has none of, or the fixed rule where it
cannot run the pick at all (a radix-8 unit)."""
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
    moma.ntt_set_schedule(q, w, n, L, None)
    got = moma.ntt_get_schedule(q, w, n, L)
    cands = moma.ntt_candidates(L, logn)
    pred = moma.costmodel_predict(np.array([moma.costmodel_features(L, logn, s) for s in cands], np.float32))
    pick = cands[int(np.argmin(pred))][:4] + (0,)
    say(f"full width {lam} bits 2^{logn}: {got}")
    assert got == (pick if pick[3] <= (2 if L <= 16 else 1) else moma.ntt_default_schedule(L, logn))
    if logn <= 14:
        x = mi.residues(f, n, L, 860, logn)
        assert (from_dev(moma.ntt_fwd(to_dev(x), q, w)) == oracle.ntt_radix2(q, L, w, x)).all()
