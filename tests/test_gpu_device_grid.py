"""Frames whose bounds and grid stay on the device (one block for the smallest,
a last-block reduction for the others, one wait at the end) against the same
frames through the host's grid (a context with stage timing): every output
bit for bit, at the sizes where the launches change and for every kind of
box, and the errors, which must leave the outputs untouched."""
import math

import numpy as np
import pytest

from paper_1603_05143_amd import ptm

pytestmark = pytest.mark.gpu


def _frame(n, kind):
    rng = np.random.default_rng(n)
    side = (n / 0.08) ** (1 / 3)
    if kind == "flat":  # an open axis without extent
        pos = rng.random((n, 3)) * [side, side, 0.0]
        return pos, np.zeros(3)
    pos = rng.random((n, 3)) * side
    box = {"periodic": [side] * 3, "open": [0.0] * 3, "mixed": [side, 0.0, side]}[kind]
    if kind != "periodic":
        pos -= 3.0 * side
    return pos, np.array(box)


def _run(torch, pos, box, flags, topological, noalloc=False, out=None):
    c = ptm.Classifier(device=0, topological=topological, flags=flags)
    try:
        d = torch.from_numpy(np.ascontiguousarray(pos)).to("cuda:0")
        out = out if out is not None else c.alloc_outputs(len(pos), "cuda:0", knn=True, derived=True)
        torch.cuda.synchronize()
        call = ptm.ptm_classify_noalloc if noalloc else ptm.ptm_classify
        st = call(c.ctx, d.data_ptr(), None, box, len(pos), ptm.PTM_ALL, math.inf, c.outputs_struct(out))
        torch.cuda.synchronize()
        return st, {k: v.cpu().numpy() for k, v in out.items()}
    finally:
        c.close()


@pytest.mark.parametrize("topological", [False, True], ids=["euclidean", "topological"])
@pytest.mark.parametrize("kind", ["periodic", "open", "mixed", "flat"])
@pytest.mark.parametrize("n", [1, 15, 200, 1023, 4096, 4097, 16384, 16385, 70001])
def test_device_grid_equals_host_grid(n, kind, topological):
    import torch
    if kind != "open" and n < 1000:
        kind = "open"  # (smaller boxes fail the periodic-box rule)
    pos, box = _frame(n, kind)
    print(f"[grid] n={n} {kind} topological={topological}", flush=True)
    st0, want = _run(torch, pos, box, ptm.PTM_F_PROFILE, topological)
    assert st0 == ptm.PTM_OK
    for noalloc in (False, True) if n <= ptm.PTM_NOALLOC_MAX_ATOMS else (False,):
        st, got = _run(torch, pos, box, 0, topological, noalloc)
        assert st == ptm.PTM_OK
        for k in want:
            assert np.array_equal(want[k].view(np.uint8), got[k].view(np.uint8)), (k, noalloc)


@pytest.mark.parametrize("n", [300, 9000, 40000])
@pytest.mark.parametrize("what", ["nan", "inf", "box"])
def test_errors_write_nothing(n, what):
    import torch
    pos, box = _frame(n, "periodic" if what != "inf" else "open")
    if what == "box":
        pos, box = pos * [1, 1, 1e-3], box * [1, 1, 1e-3]
    else:
        pos[n // 2, 1] = math.nan if what == "nan" else -math.inf
    out = ptm.Classifier.alloc_outputs(n, "cuda:0", knn=True, derived=True)
    for t in out.values():
        t.fill_(77)
    st, got = _run(torch, pos, box, 0, False, out=out)
    assert st == (ptm.PTM_E_BOX if what == "box" else ptm.PTM_E_INVALID)
    assert all((v == 77).all() for v in got.values())
    # the context state behind it serves the next frame
    good, gbox = _frame(n, "periodic")
    c = ptm.Classifier(device=0)
    try:
        for p, b in ((pos, box), (good, gbox)):
            d = torch.from_numpy(np.ascontiguousarray(p)).to("cuda:0")
            torch.cuda.synchronize()
            st = ptm.ptm_classify(c.ctx, d.data_ptr(), None, b, n, ptm.PTM_ALL, math.inf, c.outputs_struct(out))
        assert st == ptm.PTM_OK
    finally:
        c.close()


@pytest.mark.parametrize("n,side,all_exact", [(300, None, True), (16384, None, True), (16385, None, False),
                                              (17000, 10.3, True)])
def test_work_counts_name_the_search(n, side, all_exact):
    """knn_exact of the work counts: every atom where the wave-per-atom search
    runs alone (small frames, a periodic axis of fewer than five cells),
    otherwise what the other one leaves."""
    import torch
    pos, box = _frame(n, "open" if n < 1000 else "periodic")
    if side:  # thin in z
        wide = (n / 0.08 / side) ** 0.5
        pos, box = np.random.default_rng(n).random((n, 3)) * [wide, wide, side], np.array([wide, wide, side])
    c = ptm.Classifier(device=0, flags=ptm.PTM_F_PROFILE)
    try:
        c.classify(torch.from_numpy(np.ascontiguousarray(pos)).to("cuda:0"), box)
        info = ptm.ptm_frame_info(c.ctx)
    finally:
        c.close()
    print(f"[info] n={n} {info}", flush=True)
    assert (info["knn_exact"] == n) == all_exact and info["knn_exact"] <= n
