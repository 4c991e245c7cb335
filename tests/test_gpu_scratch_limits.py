"""Frames that fit the memory that is left with their own cell grid but not
with the largest one that their atoms could have: classified as with memory to
spare, call after call, and refused (nothing written) where their own grid does
not fit either."""
import ctypes as C
import math

import numpy as np
import pytest

from paper_1603_05143_amd import ptm

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("topological", [False, True], ids=["euclidean", "topological"])
@pytest.mark.parametrize("n", [3000, 50000])
def test_own_grid_fits(n, topological):
    import torch
    side = (n / 0.08) ** (1 / 3)
    pos = torch.from_numpy(np.random.default_rng(n).random((n, 3)) * side).to("cuda:0")
    box = np.array([side] * 3)
    limit = ptm.lib().ptm_selftest_scratch_limit
    limit.argtypes = [C.c_void_p, C.c_int64]
    c = ptm.Classifier(device=0, topological=topological)
    try:
        want = c.classify(pos, box, knn=True)
    finally:
        c.close()
    # bytes of an atom beyond its cells, and of the cells of both grids
    atom = 464 + (636 if topological else 0)
    own, largest = 8 * 1.5 * n, 8 * (4 * n + 4096)
    out = ptm.Classifier.alloc_outputs(n, "cuda:0", knn=True)
    for t in out.values():
        t.fill_(77)
    for room, fits in ((atom * n + 0.5 * (own + largest), True), (0.5 * atom * n, False)):
        c = ptm.Classifier(device=0, topological=topological)
        try:
            assert limit(c.ctx, int(room)) == ptm.PTM_OK
            for call in range(3):
                print(f"[scratch] n={n} topological={topological} room={room:.0f} call {call}", flush=True)
                st = ptm.ptm_classify(c.ctx, pos.data_ptr(), None, box, n, ptm.PTM_ALL, math.inf,
                                      c.outputs_struct(out))
                torch.cuda.synchronize()
                if fits:
                    assert st == ptm.PTM_OK and ptm.ptm_last_error(c.ctx) == ""
                    assert all(torch.equal(out[k].view(torch.uint8), want[k].view(torch.uint8)) for k in want)
                else:
                    assert st == ptm.PTM_E_NOMEM and "allocation" in ptm.ptm_last_error(c.ctx)
                    assert all(bool((t == 77).all()) for t in out.values())
        finally:
            c.close()
        for t in out.values():
            t.fill_(77)
