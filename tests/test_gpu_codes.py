"""Hull codes on the device against the oracle's own canonical form: isolated
clusters about the points of each template, in random rotations and vertex
orders, with noise up to where hulls of no template are common.  Their
vertices of minimum degree, where the code starts, have degree 3, 4 and 5.
Types and neighbour maps (the code's labelling) are compared exactly."""
import numpy as np
import pytest

from paper_1603_05143_amd import ptm, synthetic as S
from parity_util import TOL32, TOL64, compare

CLUSTERS = 150


def clusters(oracle_lib, t, noise):
    """Cluster centres first, then their neighbours, cluster by cluster."""
    rng = np.random.default_rng(100 * t + int(1000 * noise))
    w = np.asarray(oracle_lib.template(t)["w"])
    w = w / np.linalg.norm(w, axis=1).min()
    rot = S.random_rotations(rng, CLUSTERS)
    pts = np.einsum("cij,kj->cki", rot, w)
    pts = np.stack([p[rng.permutation(len(w))] for p in pts]) + rng.normal(scale=noise, size=pts.shape)
    centres = 40.0 * np.stack(np.meshgrid(*[np.arange(6)] * 3, indexing="ij"), -1).reshape(-1, 3)[:CLUSTERS]
    pos = np.concatenate([centres, (pts + centres[:, None]).reshape(-1, 3)])
    return np.ascontiguousarray(pos), pts


def test_inputs_reach_every_start(oracle_lib):
    seen = set()
    for t in range(5):
        for noise in (0.02, 0.08, 0.16):
            for p in clusters(oracle_lib, t, noise)[1]:
                ok, tris = oracle_lib.hull(p)
                if ok:
                    seen.add((len(p), int(np.bincount(np.asarray(tris).ravel()).min())))
    assert seen >= {(6, 4), (12, 3), (12, 4), (12, 5), (14, 3), (14, 4)}, seen


@pytest.mark.gpu
@pytest.mark.parametrize("precision", [ptm.PTM_FP64, ptm.PTM_FP32_MIXED], ids=["fp64", "fp32mixed"])
@pytest.mark.parametrize("noise", [0.02, 0.08, 0.16])
@pytest.mark.parametrize("t", range(5))
def test_codes(oracle_lib, t, noise, precision):
    import torch
    pos, _ = clusters(oracle_lib, t, noise)
    print(f"[codes] template {t} noise {noise} n={len(pos)}", flush=True)
    ref = oracle_lib.classify(pos, np.zeros(3))
    c = ptm.Classifier(device=0, precision=precision)
    try:
        out = c.classify(torch.from_numpy(pos).to("cuda:0"), np.zeros(3), knn=True)
        torch.cuda.synchronize()
        got = {k: v.cpu().numpy() for k, v in out.items()}
    finally:
        c.close()
    compare(got, ref, tol=TOL64 if precision == ptm.PTM_FP64 else TOL32)
