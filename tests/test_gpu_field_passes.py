"""The field and diagnostic passes over segments of other lengths.  A
segment's rows do not enter the arithmetic of a node, so fields and
populations are equal whatever the tile; the sums differ only in their
order, and lbm_reduce (which writes no field) is held against sums over the
fields: 1e-12 in FP64, 1e-5 in FP32 and 16-bit storage (FP32 partial sums
over at most 64 rows and a workgroup: 2^-24 times a few hundred terms)."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu


# one strip and one short segment; remainders of 4 rows; two and three strips;
# taller than one workgroup per compute unit at 4 rows
@pytest.mark.parametrize("nx,ny", [(9, 9), (50, 37), (252, 12), (253, 41), (600, 90), (31, 1301)])
@pytest.mark.parametrize("storage", [0, 1, 2, 3])
def test_fields_and_sums(lbm_mod, nx, ny, storage):
    wl = W.random_small(nx + ny, nx, ny, 3, n_blobs=4 if nx > 20 and ny > 20 else 0)
    base = lbm_mod.lattice_from_workload(wl, storage)
    base.step(4)
    f = base.get_fields()
    fluid = wl.solid == 0
    r = base.reduce()
    tol = 1e-12 if storage == 0 else 1e-5
    for q in (0, 1):
        want = np.sum(f[q][fluid])
        assert abs(r[q] - want) <= tol * abs(want)
    for tile in ((256, 64, 2), (128, 7, 0), (64, 1, 0)):
        g = lbm_mod.lattice_from_workload(wl, storage)
        g.set_tile(*tile)
        g.step(4)
        for a, b in zip(g.get_fields(), f):
            assert np.array_equal(a, b, equal_nan=True)
        s = g.reduce()
        assert np.all(np.abs(s[:2] - r[:2]) <= tol * np.abs(r[:2]))
        assert np.array_equal(s[4:], r[4:])  # maxima, minima and a count


# a corner of one 16 x 4 x 4 brick, remainders in each axis; small bricks for
# the steps only; the default brick for everything
@pytest.mark.parametrize("nx,ny,nz", [(9, 9, 9), (17, 13, 18), (96, 81, 97), (97, 121, 122)])
@pytest.mark.parametrize("storage", [0, 1, 2])
def test_small_bricks_and_sums_3d(lbm_mod, nx, ny, nz, storage):
    wl = W.random_small3d(nx + ny, nx, ny, nz, 1 | 2 | 4, n_blobs=2)
    tol = 1e-12 if storage == 0 else 1e-5
    base = lbm_mod.lattice3d_from_workload(wl, storage)
    g = lbm_mod.lattice3d_from_workload(wl, storage)
    g.set_tile(32, 8, 4, 1)
    for q in (base, g):
        q.step(3)
    f, h = base.get_fields(), g.get_fields()
    for a, b in zip(f, h):
        assert np.array_equal(a, b)
    r = base.reduce()
    fluid = wl.solid == 0
    for q in (0, 1):
        want = np.sum(f[q][fluid])
        assert abs(r[q] - want) <= tol * abs(want)
    u = np.sqrt(f[2] ** 2 + f[3] ** 2 + f[4] ** 2)
    assert abs(r[5] - u.max()) <= 1e-12 * u.max()
    assert r[6] == f[0][fluid].min() and r[7] == f[0][fluid].max() and r[8] == 0
