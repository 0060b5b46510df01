"""Small lattices run in bricks of fused steps until a tile is set: bitwise
equal to one step per launch in marching strips, at the brick plan's edges
(lattices smaller than a brick, exactly one, ragged, and each region and
number of steps that the plan chooses), with walls, periodic images, open
edges, sliding walls and diagnostics on the way.  No tolerance: the bricks
inline the strips' own arithmetic."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu


def _pair(lbm_mod, wl, storage, pops=None, diag=0):
    out = []
    for tile in (None, (256, 16, 0)):
        g = lbm_mod.lattice_from_workload(wl, storage)
        if pops is not None:
            g.set_populations(pops)
        if tile:
            g.set_tile(*tile)
        g.set_diag_interval(diag)
        out.append(g)
    return out


def _same(a, b):
    assert np.array_equal(a.get_populations(), b.get_populations())


# (nx, ny): below one brick, one brick of 4 steps (10), of 1 step in 32 x 32
# (28) and one more, ragged; 3 steps (170 x 150), 2 steps (300 x 210), single
# steps in 32 x 16 or two in 32 x 32 (450 x 333)
SIZES = [(5, 5), (10, 10), (28, 28), (29, 57), (170, 150), (300, 210), (450, 333)]


@pytest.mark.parametrize("storage", [0, 1, 2, 3])
@pytest.mark.parametrize("flags", [0, 1, 3])
@pytest.mark.parametrize("nx,ny", SIZES)
def test_bricks_equal_strips(lbm_mod, nx, ny, flags, storage):
    if nx * ny > 1000:
        wl = W.random_small(nx + flags, nx, ny, flags, n_blobs=25)
    else:
        wl = W.random_small(nx + flags, nx, ny, flags, n_blobs=0, drop=False)
    a, b = _pair(lbm_mod, wl, storage, W.random_populations(7, wl, 0.1))
    for n in (1, 7, 2, 5):  # odd counts, and runs longer than one launch
        a.step(n)
        b.step(n)
        _same(a, b)


@pytest.mark.parametrize("storage", [0, 1, 2, 3])
@pytest.mark.parametrize("wl", [W.obstacle_drop(90, 40, side=8, centre=(35.0, 20.0), r_drop=7.0, drop_centre=(16.0, 20.0)),
                                W.obstacle_drop(), W.obstacle_drop(700, 300, side=50, centre=(244.0, 150.0), r_drop=50.0,
                                                                   drop_centre=(110.0, 150.0)), W.cocurrent("couette")],
                         ids=["obstacle-small", "obstacle", "obstacle-large", "couette"])
def test_open_and_moving_boundaries(lbm_mod, wl, storage):
    a, b = _pair(lbm_mod, wl, storage)
    for n in (1, 6, 5):
        a.step(n)
        b.step(n)
        _same(a, b)


@pytest.mark.parametrize("every", [1, 3, 10])
def test_diagnostics_on_the_way(lbm_mod, every):
    wl = W.flat_drop()
    a, b = _pair(lbm_mod, wl, lbm_mod.F32, diag=every)
    for n in (4, 9, 8):
        a.step(n)
        b.step(n)
        _same(a, b)
        (da, ta), (db, tb) = a.get_diag(), b.get_diag()
        assert ta == tb and np.max(np.abs(da - db)) <= 1e-12 * np.max(np.abs(db))


def test_a_set_tile_marches_and_tuning_keeps_the_state(lbm_mod):
    wl = W.flat_drop()
    a, b = _pair(lbm_mod, wl, lbm_mod.F32)
    assert a.get_tile() == (128, 24, 10)
    a.step(5)
    a.autotune(2)
    a.step(6)
    b.step(11)
    _same(a, b)


def test_tuning_reports_the_fastest_tile(lbm_mod):
    """A lattice that is faster in bricks stays in them when tuned, and the tile
    that tuning reports is the fastest of the tiles, not the default: the droplet's
    three workgroups of 24 rows lose to shorter segments by far more than noise."""
    wl = W.flat_drop()
    a, b = _pair(lbm_mod, wl, lbm_mod.F32)
    tile = a.autotune(8)
    assert tile == a.get_tile() and tile != (128, 24, 10) and tile[1] != 24
    b.set_tile(*tile)
    for q in (a, b):
        q.step(9)
    _same(a, b)
