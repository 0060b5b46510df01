"""Large outputs come through pinned slots and several threads: every value
where the direct copy puts it (exact), at sizes around the threshold, with
ragged last chunks, with outputs left out, from two threads at once."""
import ctypes
import threading

import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu


def _lattice(lbm_mod, nx, ny, seed):
    wl = W.random_small(seed, nx, ny, 3, n_blobs=4)
    g = lbm_mod.lattice_from_workload(wl, lbm_mod.F64)
    return g, wl


@pytest.mark.parametrize("nx,ny", [(1000, 786), (1000, 787), (1201, 903)])
def test_fields_and_windows_agree(lbm_mod, nx, ny):
    # the rows' windows are small copies, the whole lattice a large one
    g, wl = _lattice(lbm_mod, nx, ny, nx)
    g.step(2)
    whole = g.get_populations()
    for y0, h in ((0, 3), (ny // 2, 2), (ny - 3, 3)):
        assert np.array_equal(whole[:, :, y0:y0 + h], g.get_populations_window(0, y0, nx, h))
    r1, r2, ux, uy = g.get_fields()
    fluid = wl.solid == 0
    assert np.array_equal(r1[fluid], _sum(whole[0])[fluid]) and not r1[~fluid].any()
    only = np.empty_like(uy)
    lbm_mod._check(g.h, lbm_mod.load_library().lbm_get_fields(g.h, None, None, None, only.ctypes.data_as(ctypes.c_void_p)))
    assert np.array_equal(only, uy)


def _sum(f):
    s = f[0].copy()
    for i in range(1, 9):
        s += f[i]
    return s


def test_two_threads(lbm_mod):
    lats = [_lattice(lbm_mod, 1300, 900, s)[0] for s in (1, 2)]
    want = [g.get_fields() for g in lats]
    got = [None, None]

    def go(i):
        for _ in range(3):
            got[i] = lats[i].get_fields()

    th = [threading.Thread(target=go, args=(i,)) for i in range(2)]
    [t.start() for t in th]
    [t.join() for t in th]
    for a, b in zip(got, want):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("where", ["pinned", "device"])
def test_outputs_in_memory_that_hip_knows(lbm_mod, where):
    """Pinned and device arrays as outputs, above the threshold and below it."""
    import torch
    for nx, ny in ((1201, 903), (300, 200)):
        g, _ = _lattice(lbm_mod, nx, ny, nx)
        g.step(2)
        kw = dict(pin_memory=True) if where == "pinned" else dict(device="cuda")
        out = [torch.empty(ny, nx, dtype=torch.float64, **kw) for _ in range(4)]
        lbm_mod._check(g.h, lbm_mod.load_library().lbm_get_fields(g.h, *[ctypes.c_void_p(t.data_ptr()) for t in out]))
        torch.cuda.synchronize()
        for a, b in zip(out, g.get_fields()):
            assert np.array_equal(a.cpu().numpy(), b)
