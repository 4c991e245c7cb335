"""Misorientation at the edges of a block's round of pairs and of the grid's
stride, every type (scans over sign patterns, over elements, and none), all
signs of the products, against the oracle.  An angle is 2 atan2(|v|, |w|) of a
product of unit quaternions rounded a few times: 1e-14 plus the oracle's own
arc cosine, whose error is eps / sin(angle / 2); pairs closer than 0.02 rad
are left to the checks near zero elsewhere."""
import numpy as np
import pytest

from paper_1603_05143_amd import ptm
from oracle import derived as OD

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "misaligned"])
@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 1500])
def test_pairs(n, offset):
    import torch
    rng = np.random.default_rng(n)
    q = rng.normal(size=(2, n, 4))
    q /= np.linalg.norm(q, axis=2, keepdims=True)
    t = rng.integers(0, 6, size=n).astype(np.int8)
    want = np.array([OD.misorientation(q[0, i], q[1, i], int(t[i]) - 1) if t[i] else
                     2 * np.arccos(min(1.0, abs(OD.quat_mul(OD.conj(q[0, i]), q[1, i])[0]))) for i in range(n)])
    bufs = [torch.empty(4 * n + 1, dtype=torch.float64, device="cuda:0")[offset:offset + 4 * n] for _ in range(2)]
    for b, x in zip(bufs, q):
        b.copy_(torch.from_numpy(x.ravel()))
    dt, out = torch.from_numpy(t).cuda(), torch.full((n,), -1.0, dtype=torch.float64, device="cuda:0")
    print(f"[misorientation] n={n} offset={offset}", flush=True)
    c = ptm.Classifier(device=0)
    try:
        torch.cuda.synchronize()
        assert ptm.ptm_misorientation(c.ctx, dt.data_ptr(), bufs[0].data_ptr(), bufs[1].data_ptr(), n,
                                      out.data_ptr()) == ptm.PTM_OK
        torch.cuda.synchronize()
        got = out.cpu().numpy()
    finally:
        c.close()
    far = want > 0.02
    assert np.all(np.abs(got - want)[far] <= 1e-14 + 8 * np.finfo(float).eps / np.sin(want[far] / 2))
    assert np.all(np.abs(got - want)[~far] <= 1e-6)
