"""The lane-per-atom neighbour search (frames above 16,384 atoms) against the
oracle's, where it can go wrong: axes of 5 to 8 cells, on which ranges wrap, at
every pair of axes; rows of more atoms than a table entry or a table holds,
also across the box edge; ties that end inside and past the key list, lists
that fill up (coincident atoms); coordinates inside, around and far outside the
box, whose fixed-point steps are coarse; blocks that wrap beside blocks that do
not (the shortcut without shifts); tiles of cells that are cut short; and a
periodic axis of fewer than five cells, which the search leaves to the other
one.  Ids are compared exactly."""
import numpy as np
import pytest

from paper_1603_05143_amd import ptm, synthetic as S

pytestmark = pytest.mark.gpu
RHO = 0.08
CELL = 0.6 * (14 / (4.1887902047863905 * RHO)) ** (1 / 3)  # at that density


def _gas(n, box, seed):
    box = np.asarray(box, float)
    return np.random.default_rng(seed).random((n, 3)) * box, box


def _frame(kind):
    rng = np.random.default_rng(12)
    name, _, arg = kind.partition(":")
    if name == "cells":  # k cells on the two axes named, the rest on the third
        k, axes = float(arg[0]) + 0.4, [int(a) for a in arg[1:]]
        box = np.full(3, 17000 / RHO / (k * CELL) ** 2)
        box[axes] = k * CELL
        return _gas(17000, box, int(k))
    if name == "thin":  # four cells on one axis
        box = np.full(3, (18000 / RHO / (4.9 * CELL)) ** 0.5)
        box[int(arg)] = 4.9 * CELL
        return _gas(18000, box, 3)
    if name == "dense_row":  # 5000 atoms within one row of cells, at the edge of the box or inside
        pos, box = _gas(17000, [60.0] * 3, 4)
        line = np.c_[(0.0 if arg == "edge" else 25.0) + 8 * rng.random(5000), 20 + rng.random((5000, 2))]
        line[:, 0] = (line[:, 0] - 4.0) % 60.0
        return np.vstack([pos, line]), box
    if name == "coincident":
        return np.vstack([np.full((300, 3), 7.5), np.full((40, 3), 20.0), rng.random((18000, 3)) * 60]), np.zeros(3)
    if name == "ties":
        reps = {"sc": 27, "bcc": 21, "fcc": 17}[arg]
        f = S.perfect_crystal(arg, reps=(reps,) * 3)
        return f.positions, f.box
    if name == "unwrapped":
        pos, box = _gas(20000, [62.0, 64.0, 63.0], 5)
        return pos + box * rng.integers(-3, 4, size=pos.shape), box
    if name == "far_unwrapped":  # wrapping these costs more than a fixed-point step
        pos, box = _gas(20000, [62.0, 64.0, 63.0], 6)
        return pos + box * rng.integers(-200000, 200001, size=pos.shape), box
    if name == "tiles":  # 11 x 19 rows of cells: whole, partial and corner tiles
        return _gas(24000, [24000 / RHO / (11.3 * 19.2 * CELL**2), 11.3 * CELL, 19.2 * CELL], 8)
    if name == "slab":
        return _gas(20000, [60.0, 60.0, 69.0], 9)[0], np.array([60.0, 60.0, 300.0])
    assert name == "open"
    return _gas(20000, [62.0, 64.0, 63.0], 10)[0] - 31.0, np.zeros(3)


KINDS = [f"cells:{k}{a}" for k in (5, 6, 7, 8) for a in ("01", "02", "12")] + [
    "thin:0", "thin:2", "dense_row:inside", "dense_row:edge", "coincident", "ties:sc", "ties:bcc", "ties:fcc",
    "unwrapped", "far_unwrapped", "tiles", "slab", "open"]


@pytest.mark.parametrize("topological", [False, True], ids=["euclidean14", "topological18"])
@pytest.mark.parametrize("kind", KINDS)
def test_neighbours(oracle_lib, kind, topological):
    import torch
    pos, box = _frame(kind)
    pos = np.ascontiguousarray(pos)
    assert len(pos) > 16384
    print(f"[knn lanes] {kind} n={len(pos)} box={box} topological={topological}", flush=True)
    ids, _, _, _, box_ok = oracle_lib.neighbours(pos, box, K=18 if topological else 14)
    c = ptm.Classifier(device=0, topological=topological)
    try:
        dpos = torch.from_numpy(pos).to("cuda:0")
        if not box_ok:
            with pytest.raises(ptm.PTMError) as e:
                c.classify(dpos, box, knn=True)
            assert e.value.status == ptm.PTM_E_BOX
            return
        got = c.classify(dpos, box, knn=True)["knn"].cpu().numpy()
    finally:
        c.close()
    bad = np.flatnonzero((got != ids[:, :14]).any(1))
    assert bad.size == 0, (len(bad), bad[:5], got[bad[:1]], ids[bad[:1]])
