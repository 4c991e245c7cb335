"""The exact predicates in fixed point (and their fall-back on expansions for
points that do not fit), through the library's host self-checks, against the
oracle's exact predicates: noise-free rotated lattice shells (coplanar up to
the rounding of the coordinates), exactly degenerate integer sets, sets whose
coordinates span more than the fixed-point range, and extreme magnitudes.
The GPU test classifies noise-free crystals, whose every atom needs them."""
import ctypes as C
import math

import numpy as np
import pytest

from paper_1603_05143_amd import ptm, synthetic as S


def _rot(rng):
    return S.random_rotations(rng, 1)[0]


def _sets(kind, rng):
    """Four points, many of them within a few ulps of coplanar."""
    shell = np.array([[x, y, 0] for x in (1, -1) for y in (1, -1)], float) * 1.8075
    if kind == "rotated":  # the four corners of a square facet, coordinates rounded
        q = shell @ _rot(rng).T + 57.3 * rng.random(3)
        return q - q[rng.integers(4)] * rng.integers(0, 2)
    if kind == "ulp":
        q = shell @ _rot(rng).T
        q[rng.integers(4), rng.integers(3)] = np.nextafter(q[0, 0], 9.0)
        return q
    if kind == "integer":
        q = rng.integers(-2, 3, size=(4, 3)).astype(float) * 3.615
        return q
    if kind == "span":  # one coordinate far finer than the others: does not fit
        q = rng.integers(-1, 2, size=(4, 3)).astype(float)
        q[rng.integers(4), rng.integers(3)] += 2.0 ** -rng.integers(40, 75)
        q[rng.integers(4), rng.integers(3)] = 2.0 ** -rng.integers(50, 120)
        return q
    if kind == "scaled":  # any magnitude
        q = rng.integers(-3, 4, size=(4, 3)).astype(float)
        q[3] = q[0] + q[1] - q[2]
        return q * 2.0 ** rng.integers(-90, 90)
    return np.zeros((4, 3))  # "zero": all points coincide


@pytest.mark.parametrize("kind", ["rotated", "ulp", "integer", "span", "scaled", "zero"])
def test_orient_and_det3_sign(oracle_lib, kind):
    L = ptm.lib()
    rng = np.random.default_rng(len(kind))
    for _ in range(600):
        q = np.ascontiguousarray(_sets(kind, rng))
        r = rng.permutation(14)[:4].astype(np.int32)
        assert L.ptm_selftest_orient(q.ctypes.data_as(C.c_void_p), r.ctypes.data_as(C.c_void_p)) == \
            oracle_lib.orient(q, r, sos=True), (q, r)
        from fractions import Fraction as F
        a, b, c = ([F(float(x)) for x in v] for v in q[:3])
        d = (a[0] * (b[1] * c[2] - b[2] * c[1]) + a[1] * (b[2] * c[0] - b[0] * c[2]) +
             a[2] * (b[0] * c[1] - b[1] * c[0]))
        assert L.ptm_selftest_det3(q.ctypes.data_as(C.c_void_p)) == (d > 0) - (d < 0)


def _crystal(kind):
    rng = np.random.default_rng(5)
    if kind == "polycrystal":
        f = S.polycrystal(L=32.0, n_grains=3, sigma=0.0, seed=77)
        return f.positions, np.array(f.box)
    f = S.perfect_crystal(kind, reps=(6, 6, 6))
    pos = f.positions - f.box / 2
    pos = pos[(pos ** 2).sum(1) < (0.5 * f.box.min()) ** 2]
    return np.ascontiguousarray(pos @ _rot(rng).T + 41.7), np.zeros(3)  # a rotated sphere with free surfaces


@pytest.mark.gpu
@pytest.mark.parametrize("form", [ptm.PTM_FP64, ptm.PTM_FP32_MIXED], ids=["fp64", "fp32mixed"])
@pytest.mark.parametrize("kind", ["fcc", "bcc", "hcp", "sc", "polycrystal"])
def test_noise_free_crystals(oracle_lib, kind, form):
    import torch
    pos, box = _crystal(kind)
    print(f"[fixed] {kind} n={len(pos)} form={form}", flush=True)
    ref = oracle_lib.classify(pos, box)
    c = ptm.Classifier(device=0, precision=form)
    out = c.classify(torch.from_numpy(np.ascontiguousarray(pos)).to("cuda:0"), box, knn=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in out.items()}
    c.close()
    for k in ("type", "knn", "neighbours"):
        assert np.array_equal(got[k], ref[k]), (k, np.flatnonzero((got[k] != ref[k]).reshape(len(pos), -1).any(1))[:5])
    fin = np.isfinite(ref["rmsd"])
    assert np.array_equal(fin, np.isfinite(got["rmsd"]))
    tol = 1e-12 if form == ptm.PTM_FP64 else 1e-5
    assert np.max(np.abs(got["rmsd"][fin] - ref["rmsd"][fin]), initial=0.0) <= tol
    assert math.isfinite(float(got["strain"].sum()))
