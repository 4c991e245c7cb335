"""The match stage where its waves hold many atoms: 2, 32 and 64 atoms a wave
(frames above 1,024, 16,384 and 32,768 atoms), a last wave or block that is
nearly empty or one short, and several candidates an atom, so that a wave's jobs
run over many chunks of 64 and atoms straddle their boundaries.  Frames mix
perfect lattice (explicit residuals), noise (residuals from moments) and
surfaces (no candidate).  Compared with the oracle: types and neighbour maps
exactly, reals as everywhere."""
import numpy as np
import pytest

from paper_1603_05143_amd import ptm, synthetic as S
from parity_util import TOL32, TOL64, compare

pytestmark = pytest.mark.gpu


def _frame(n):
    rng = np.random.default_rng(n)
    parts = []
    for i, (kind, a, cell) in enumerate((("fcc", 3.6, 4), ("bcc", 2.9, 2), ("sc", 2.6, 1))):
        m = n // 3 + 1
        reps = int(np.ceil((1.95 * m / cell) ** (1 / 3))) + 1  # (a ball of m atoms fits)
        k = S.perfect_crystal(kind, (reps,) * 3, a=a).positions
        k = k[np.argsort(((k - k.mean(0)) ** 2).sum(1), kind="stable")[:m]]
        parts.append(k - k.mean(0) + [300.0 * i, 0, 0])
    pos = np.concatenate(parts)[:n]
    noisy = rng.random(len(pos)) < 0.7
    pos = pos + rng.normal(scale=0.06, size=pos.shape) * noisy[:, None]
    return np.ascontiguousarray(pos)


@pytest.fixture(scope="module")
def references(oracle_lib):
    done = {}

    def get(n, mask):
        if (n, mask) not in done:
            done[n, mask] = oracle_lib.classify(_frame(n), np.zeros(3), mask=mask)
        return done[n, mask]
    return get


CASES = [(n, mask) for mask in (ptm.PTM_ALL, ptm.PTM_ICO, ptm.PTM_SC | ptm.PTM_HCP)
         for n in ((1025, 2047, 20001, 32767, 32769, 33023, 33024, 33025) if mask == ptm.PTM_ALL else (1025, 33025))]


@pytest.mark.parametrize("precision", [ptm.PTM_FP64, ptm.PTM_FP32_MIXED], ids=["fp64", "fp32mixed"])
@pytest.mark.parametrize("n,mask", CASES)
def test_chunks(references, n, mask, precision):
    import torch
    pos = _frame(n)
    print(f"[match chunks] n={n} mask={mask}", flush=True)
    ref = references(n, mask)
    c = ptm.Classifier(device=0, precision=precision, flags=ptm.PTM_F_PROFILE)
    try:
        out = c.classify(torch.from_numpy(pos).to("cuda:0"), np.zeros(3), mask=mask, knn=True)
        got = {k: v.cpu().numpy() for k, v in out.items()}
        info = ptm.ptm_frame_info(c.ctx)
    finally:
        c.close()
    if mask == ptm.PTM_ALL and n > 20000:  # several candidates an atom
        assert info["pairs"] > 1.5 * n, info
    compare(got, ref, tol=TOL64 if precision == ptm.PTM_FP64 else TOL32)
