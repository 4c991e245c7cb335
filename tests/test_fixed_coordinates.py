"""Fixed-point coordinates of the neighbour search (CPU): the 32-bit difference
of two points less than three cells apart is their minimum image to within the
stated bound, in short and long boxes, open and periodic, wrapped or not, and
the steps stay as fine against a cell on the longest axes as on the shortest.
On the GPU, a wire of 3 * 10^5 cells keeps its atoms in the lane-per-atom
search."""
import ctypes as C

import numpy as np
import pytest

from paper_1603_05143_amd import ptm


def _fixed(box, mn, mx, n, x):
    coord, scale = np.zeros(3, np.int32), np.zeros(7)
    a = [np.ascontiguousarray(v, np.float64) for v in (box, mn, mx)]
    x = np.ascontiguousarray(x, np.float64)
    ok = ptm.lib().ptm_selftest_fixed(*[v.ctypes.data_as(C.c_void_p) for v in a], C.c_int64(n), 14,
                                      x.ctypes.data_as(C.c_void_p), coord.ctypes.data_as(C.c_void_p),
                                      scale.ctypes.data_as(C.c_void_p))
    assert ok
    return coord, scale[:3], scale[3:6], scale[6]


@pytest.mark.parametrize("lx", [12.0, 20.0, 40.0, 333.0, 5e3, 1e5, 2e6])
@pytest.mark.parametrize("kind", ["periodic", "open", "unwrapped"])
def test_differences_are_minimum_images(kind, lx):
    rng = np.random.default_rng(int(lx))
    L = np.array([lx, 13.0, 60.0])
    n = max(20, int(0.08 * L.prod()))
    box = np.zeros(3) if kind == "open" else L
    shift = 5.0 if kind == "unwrapped" else 0.0
    mn, mx = -shift * L - (kind == "open") * 7.0, (1 + shift) * L * (1 - 1e-15) - (kind == "open") * 7.0
    for k in range(300):
        a = mn + rng.random(3) * (mx - mn)
        if k % 3 == 0:  # at an edge of the box
            a = np.where(rng.random(3) < 0.5, mn, mx)
        ca, fix, h, err = _fixed(box, mn, mx, n, a)
        d = (2 * rng.random(3) - 1) * np.minimum(2.99 * h, 0.49 * L)
        b = a + d
        if kind == "open":
            b = np.clip(b, mn, mx)
        elif kind == "periodic":
            b = b - L * np.floor(b / L)
            b = np.minimum(b, mx)
        else:
            b = np.clip(b, mn, mx) + 0.0
        cb = _fixed(box, mn, mx, n, b)[0]
        true = b - a
        if kind != "open":
            true = true - L * np.rint(true / L)
        got = (cb.astype(np.int64) - ca.astype(np.int64)).astype(np.int32) / fix
        assert np.linalg.norm(got - true) <= err + 1e-15 * np.abs(mx).max(), (a, b, got, true, err)
    # a difference vector is off by no more than a millionth of a cell, or FP64's own grain there
    assert err <= 1e-6 * h.max() + 4e-15 * np.abs([mn, mx]).max()
    assert (2.99 * h * fix)[h < L / 6].max(initial=0) < 2**31


def _wire(n, periodic):
    """Positions, box, neighbours and the share of atoms left to the exact
    search in a gas of n atoms in a wire of 6.2 x 6.2."""
    import torch
    side = 6.2
    L = np.array([n / 0.08 / side**2, side, side])
    pos = np.ascontiguousarray(np.random.default_rng(4).random((n, 3)) * L)
    print(f"[wire] n={n} L={L} periodic={periodic}", flush=True)
    c = ptm.Classifier(device=0, flags=ptm.PTM_F_PROFILE)
    try:
        box = np.array([L[0] if periodic else 0.0, 0.0, 0.0])
        got = c.classify(torch.from_numpy(pos).to("cuda:0"), box, knn=True)["knn"].cpu().numpy()
        info = ptm.ptm_frame_info(c.ctx)
    finally:
        c.close()
    print(info, flush=True)
    return pos, L, got, info["knn_exact"] / n


@pytest.mark.gpu
@pytest.mark.parametrize("periodic", [False, True], ids=["open", "periodic"])
def test_long_wire(oracle_lib, periodic):
    # (thin: some atoms' neighbours reach past the block of cells at any length)
    short = _wire(40_000, periodic)[-1]
    pos, L, got, left = _wire(2_000_000, periodic)
    assert short < 1.0 and abs(left - short) < 0.02, (left, short)
    # a stretch at the box edge and one in the middle against the oracle
    x = pos[:, 0]
    for lo, hi in ((0.4 * L[0], 0.4 * L[0] + 3000), (-1500.0, 1500.0)):
        xs = np.where(x > L[0] / 2, x - L[0], x) if lo < 0 and periodic else x
        sel = np.flatnonzero((xs > lo) & (xs < hi))
        ids = oracle_lib.neighbours(np.ascontiguousarray(np.c_[xs[sel], pos[sel, 1:]]), np.zeros(3), K=14)[0]
        inner = np.flatnonzero((xs[sel] > lo + 50 * (lo > 0 or periodic)) & (xs[sel] < hi - 50))
        assert len(inner) > 500 and np.array_equal(got[sel[inner]], sel[ids[inner]])
