"""Neighbour search in frames that are mostly empty: atoms hundreds of
thousands of empty cells from all others, whose exact search grows its block
over the whole grid.  Ids are compared exactly with the oracle's."""
import numpy as np
import pytest

from paper_1603_05143_amd import ptm

pytestmark = pytest.mark.gpu


def _stray(n, kind):
    rng = np.random.default_rng(n)
    side = (n / 0.08) ** (1 / 3)
    pos = rng.random((n, 3)) * side
    if kind == "line":  # all cells along x
        pos[:2] = [[1e9, 0, 0], [5e8, 1, 2]]
        return pos, np.zeros(3)
    if kind == "corners":
        pos[:4] = [[1e6, 0, 0], [0, 5e5, 2], [0, -4e5, 3e5], [1e6, 5e5, 3e5]]
        return pos, np.zeros(3)
    assert kind == "periodic"
    pos[0] = [25 * side, 3e5, 12 * side]
    return pos, np.array([50 * side, 0.0, 50 * side])


@pytest.mark.parametrize("topological", [False, True], ids=["euclidean14", "topological18"])
@pytest.mark.parametrize("kind", ["line", "corners", "periodic"])
@pytest.mark.parametrize("n", [900, 20000])
def test_stray_atoms(oracle_lib, n, kind, topological):
    import torch
    pos, box = _stray(n, kind)
    print(f"[sparse] {kind} n={n} topological={topological}", flush=True)
    ids, _, _, _, box_ok = oracle_lib.neighbours(pos, box, K=18 if topological else 14)
    c = ptm.Classifier(device=0, topological=topological)
    try:
        dpos = torch.from_numpy(np.ascontiguousarray(pos)).to("cuda:0")
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
