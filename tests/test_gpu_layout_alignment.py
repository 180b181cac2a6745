"""GPU parity of pack and unpack where the element-major side is and is not
aligned to 16 bytes, for whole blocks of 256 elements, a ragged last one and
less than a block."""
import numpy as np
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("limbs", [2, 3, 8, 13, 31, 32])
@pytest.mark.parametrize("offset", [0, 1, 2, 4])
def test_element_major_side_at_any_alignment(limbs, offset):
    import paper_2501_07535_amd as moma
    rng = np.random.default_rng(limbs)
    for n in (5, 256, 512, 777):
        say(f"limbs={limbs} offset={offset} n={n}")
        host = rng.integers(-2 ** 31, 2 ** 31, size=(n, limbs), dtype=np.int64).astype(np.int32)
        flat = torch.zeros(n * limbs + offset, dtype=torch.int32, device="cuda:0")
        e = flat[offset:].view(n, limbs)
        e.copy_(torch.from_numpy(host))
        p = moma.pack(e)
        assert (p.cpu().numpy() == host.T).all()
        back = torch.zeros_like(flat)
        moma.unpack(p, out=back[offset:].view(n, limbs))
        assert (back[offset:].cpu().numpy().reshape(n, limbs) == host).all() and (back[:offset] == 0).all()
