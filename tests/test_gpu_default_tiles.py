"""The tile the library picks where the caller sets none: segments shortened on
lattices that would leave SIMDs idle, other strips at relaxation time 1, one or
two steps per launch with open edges by size.  Populations do not depend on the
tile (bitwise), so each choice is held against a tile set by hand."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu


def _workload(kind, nx, ny):
    if kind == "walls":
        return W.random_small(nx, nx, ny, 1, n_blobs=40, walls=True)
    return W.obstacle_drop(nx, ny, side=40, centre=(nx / 3.0, ny / 2.0), r_drop=60.0, drop_centre=(nx / 6.0, ny / 2.0))


# past the lattices that run in bricks: rows cut to about 14, to 26, a width of
# a few strips, one segment per SIMD and a few more, and (open, 16 million nodes) three rounds of wavefronts
@pytest.mark.parametrize("kind,nx,ny,storage,tau", [
    ("walls", 1100, 800, 1, 0.9), ("walls", 1100, 800, 1, 1.0), ("walls", 1700, 720, 2, 0.9), ("walls", 1700, 720, 3, 1.0),
    ("walls", 300, 4001, 0, 0.9), ("walls", 300, 4001, 0, 1.0), ("walls", 1600, 1700, 0, 0.9), ("open", 1801, 701, 2, 1.0), ("open", 1801, 701, 1, 1.0),
    ("open", 8201, 1991, 3, 1.0),
])
def test_default_tile_equals_a_set_one(lbm_mod, kind, nx, ny, storage, tau):
    wl = _workload(kind, nx, ny)
    wl.tau = tau
    g = lbm_mod.lattice_from_workload(wl, storage)
    ref = lbm_mod.lattice_from_workload(wl, storage)
    ref.set_tile(128, 16, 2)
    for q in (g, ref):
        q.step(1)
        q.step(4)
    x0, w = nx // 3, min(nx // 3, 400)
    assert np.array_equal(g.get_populations_window(x0, 0, w, ny), ref.get_populations_window(x0, 0, w, ny))
    for a, b in zip(g.get_fields(), ref.get_fields()):
        assert np.array_equal(a, b)


# a few rows, so wide that one row of segments is more wavefronts than the
# registers hold at once (FP64 60 000 x 10 steps in bricks, its field passes march)
@pytest.mark.parametrize("nx,ny,storage,tau", [(60000, 40, 0, 0.9), (60000, 10, 0, 0.9), (130000, 20, 0, 1.0),
                                               (130000, 16, 1, 0.85), (200000, 20, 1, 1.0), (180000, 30, 2, 0.9),
                                               (250000, 30, 3, 1.0)])
def test_wide_lattices_of_few_rows(lbm_mod, nx, ny, storage, tau):
    wl = W.random_small(nx, nx, ny, 1, n_blobs=20, walls=True, drop=False)
    wl.tau = tau
    g = lbm_mod.lattice_from_workload(wl, storage)
    ref = lbm_mod.lattice_from_workload(wl, storage)
    ref.set_tile(128, 16, 2)
    for q in (g, ref):
        q.step(1)
        q.step(4)
    for a, b in zip(g.get_fields(), ref.get_fields()):
        assert np.array_equal(a, b)
    r, s = g.reduce(), ref.reduce()
    assert np.array_equal(r[4:], s[4:])  # maxima, minima and a count
    x0, w = nx // 3, 5000
    assert np.array_equal(g.get_populations_window(x0, 0, w, ny), ref.get_populations_window(x0, 0, w, ny))


# a step that records runs alone in a tile of its own
@pytest.mark.parametrize("kind,nx,ny,storage", [("walls", 1100, 800, 1), ("walls", 1700, 720, 2), ("walls", 300, 4001, 0),
                                                ("open", 1801, 701, 1), ("open", 1801, 701, 3), ("open", 1801, 701, 0),
                                                ("walls", 100, 60, 1), ("open", 350, 150, 2)])
def test_recording_steps_by_default(lbm_mod, kind, nx, ny, storage):
    wl = W.obstacle_drop() if kind == "open" and nx == 350 else _workload(kind, nx, ny)
    wl.tau = 0.9
    g = lbm_mod.lattice_from_workload(wl, storage)
    ref = lbm_mod.lattice_from_workload(wl, storage)
    ref.set_tile(128, 16, 2)
    for q in (g, ref):
        q.set_diag_interval(1)
        q.step(1)
        q.step(4)
    (d, t), (r, _) = g.get_diag(), ref.get_diag()
    tol = 1e-12 if storage == 0 else 1e-5  # sums in another order (FP32 partial sums below FP64)
    assert t == 4 and np.array_equal(d[4:], r[4:])  # maxima, minima and a count
    assert np.all(np.abs(d[:2] - r[:2]) <= tol * np.abs(r[:2]))
    assert np.all(np.abs(d[2:4] - r[2:4]) <= tol * (r[0] + r[1]) * r[4])
    for a, b in zip(g.get_fields(), ref.get_fields()):
        assert np.array_equal(a, b)
