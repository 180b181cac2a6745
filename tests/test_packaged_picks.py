"""The packaged cost model on the CPU: its first choice at every recorded size is
the recorded one, and the recorded choices cost little against the fastest shape
measured at each size: 3.2% on average, as the model did that it stands in for
on the kernels of its time, and at no range of sizes twice that."""
import json
import math
import os
import sys

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def _record():
    with open(os.path.join(ROOT, "profiles", "costmodel_picks.json")) as fh:
        return json.load(fh)["by_shape"]


def _mean(values):
    return math.expm1(sum(math.log1p(v) for v in values) / len(values))


def test_recorded_regret():
    rec = {tuple(int(v) for v in k.split(",")): v["regret"] for k, v in _record().items()}
    main = {k: v for k, v in rec.items() if k[1] >= 10}
    assert {(L, n) for L in range(2, 33) for n in range(10, 25)} <= set(main)
    assert _mean(main.values()) <= 0.032
    assert max(rec.values()) <= 0.35
    for low, high in ((6, 9), (10, 13), (14, 17), (18, 21), (22, 26)):
        assert _mean([v for (L, n), v in rec.items() if low <= n <= high]) <= 0.064, (low, high)


def test_record_is_the_packaged_models():
    import paper_2501_07535_amd as moma
    from paper_2501_07535_amd import tuning
    fm, fs, tm, ts, w = tuning.read_model(moma.COSTMODEL_PATH)
    w1, b1, w2, b2, w3, b3 = tuning._layers(w)
    rec = _record()
    for k in sorted(rec)[::7]:
        L, logn = (int(v) for v in k.split(","))
        cands = moma.ntt_candidates(L, logn)
        x = (np.array([moma.costmodel_features(L, logn, s) for s in cands], np.float32) - fm) / fs
        h = np.maximum(np.maximum(x @ w1.T + b1, 0) @ w2.T + b2, 0)
        pred = (h @ w3.T + b3)[:, 0]
        got = pred[cands.index(tuple(rec[k]["pick"]))]
        assert got <= pred.min() + 1e-4, k  # (single precision, summed in another order)
