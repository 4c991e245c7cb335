"""Frames whose extents leave no cell grid of the size the arrays are laid out
for: edges so different that the coarsest grid in x is one cell in y and z and
still too long, volumes that underflow, differences that overflow.  The grid
says so (CPU), and every entry point refuses the frame as the host's grid
always did, writes nothing and serves the next frame (GPU)."""
import ctypes as C
import math

import numpy as np
import pytest

from paper_1603_05143_amd import ptm

# per-axis extents of an open frame
BAD = {"thin": [1e3, 1e-40, 1e-40], "tiny": [1e-103, 1e-103, 1e-103], "overflow": [math.inf, 10.0, 10.0]}
GOOD = {"cube": [20.0, 20.0, 20.0], "flat": [1e3, 1e-160, 1e-170], "huge": [1e120, 1e120, 1e120],
        "needle": [1e9, 1.0, 1.0]}
SIZES = [1, 500, 4096, 4097, 20000]


def _grid(ext, n, kn=14):
    half = np.array([9.5e307 if math.isinf(e) else 0.5 * e for e in ext])
    out = np.zeros(4, np.int64)
    args = [np.ascontiguousarray(a, np.float64) for a in ([0.0] * 3, -half, half)]
    fits = ptm.lib().ptm_selftest_grid(*[a.ctypes.data_as(C.c_void_p) for a in args], C.c_int64(n), kn,
                                       out.ctypes.data_as(C.c_void_p))
    return fits, [int(x) for x in out]


@pytest.mark.parametrize("n", SIZES + [300000, 2000000, 2**31 - 2])
@pytest.mark.parametrize("name", list(BAD) + list(GOOD))
def test_grid_says_whether_it_fits(name, n):
    fits, (nx, ny, nz, cells) = _grid({**BAD, **GOOD}[name], n)
    assert cells == nx * ny * nz and min(nx, ny, nz) >= 1
    assert fits == (cells <= 4 * n + 4096)
    if name in GOOD or (name == "thin" and n >= 300000):
        assert fits
    elif name == "overflow":
        assert not fits  # at any number of atoms: no cell has an edge
    elif n <= 20000:
        assert not fits


def _frame(name, n):
    rng = np.random.default_rng(n)
    ext = np.array(BAD[name])
    half = np.where(np.isinf(ext), 9.5e307, 0.5 * ext)
    pos = (2 * rng.random((n, 3)) - 1) * half
    pos[0], pos[-1] = -half, half
    return np.ascontiguousarray(pos)


@pytest.mark.gpu
@pytest.mark.parametrize("topological", [False, True], ids=["euclidean", "topological"])
@pytest.mark.parametrize("name", list(BAD))
@pytest.mark.parametrize("n", SIZES[1:])
def test_refused(n, name, topological):
    import torch
    pos = _frame(name, n)
    assert _grid(BAD[name], n, 18 if topological else 14)[0] == 0
    print(f"[grid limits] {name} n={n}", flush=True)
    good = np.random.default_rng(1).random((n, 3)) * (n / 0.08) ** (1 / 3)
    c = ptm.Classifier(device=0, topological=topological)
    try:
        dpos, dgood = (torch.from_numpy(p).to("cuda:0") for p in (pos, good))
        out = c.alloc_outputs(n, "cuda:0", knn=True, derived=True)
        for t in out.values():
            t.fill_(77)
        torch.cuda.synchronize()
        for call, want in ((ptm.ptm_classify, ptm.PTM_E_NOMEM), (ptm.ptm_classify_noalloc, ptm.PTM_E_TOO_LARGE)):
            st = call(c.ctx, dpos.data_ptr(), None, np.zeros(3), n, ptm.PTM_ALL, math.inf, c.outputs_struct(out))
            torch.cuda.synchronize()
            assert st == want, (st, ptm.ptm_last_error(c.ctx))
            assert "cell grid" in ptm.ptm_last_error(c.ctx)
            assert all(bool((t == 77).all()) for t in out.values())
        st = ptm.ptm_classify(c.ctx, dgood.data_ptr(), None, np.zeros(3), n, ptm.PTM_ALL, math.inf,
                              c.outputs_struct(out))
        assert st == ptm.PTM_OK
    finally:
        c.close()


@pytest.mark.gpu
@pytest.mark.parametrize("flags", [0, ptm.PTM_F_PERSISTENT], ids=["streams", "persistent"])
def test_serving_refuses(flags):
    import torch
    n = 500
    good = np.random.default_rng(1).random((n, 3)) * (n / 0.08) ** (1 / 3)
    c = ptm.Classifier(device=0, flags=flags)
    try:
        out = c.alloc_outputs(n, "cuda:0", knn=True)
        for t in out.values():
            t.fill_(77)
        for name in list(BAD) + [None]:
            pos = torch.from_numpy(good if name is None else _frame(name, n)).to("cuda:0")
            torch.cuda.synchronize()
            print(f"[grid limits] serving {name}", flush=True)
            st, ticket = ptm.ptm_submit(c.ctx, pos.data_ptr(), None, np.zeros(3), n, ptm.PTM_ALL, math.inf,
                                        c.outputs_struct(out))
            if st == ptm.PTM_OK:
                st, _ = ptm.ptm_wait(c.ctx, ticket, 20_000_000)
            torch.cuda.synchronize()
            if name is None:
                assert st == ptm.PTM_OK
            else:
                assert st == (ptm.PTM_E_NOMEM if flags else ptm.PTM_E_DEVICE), st
                assert "cell grid" in ptm.ptm_last_error(c.ctx)
                assert all(bool((t == 77).all()) for t in out.values())
    finally:
        c.close()
