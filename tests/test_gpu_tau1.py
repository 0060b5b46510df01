"""At relaxation time 1 the marching kernels keep momenta instead of
populations.  FP64 against the oracle to 1e-12 (the library's bound for FP64
everywhere), and every storage against the bricks and the diagnostic passes,
which keep the populations: equal values (their factor 1 - omega is zero, so
no tolerance)."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu

TILES = [(64, 8, 0), (64, 24, 8), (128, 16, 10), (256, 0, 0), (256, 16, 10)]


def _case(kind):
    if kind == "walls":
        wl = W.random_small(5, 75, 41, 1, n_blobs=9, walls=True)
    elif kind == "periodic":
        wl = W.random_small(6, 61, 38, 3, n_blobs=5)
    elif kind == "open":
        wl = W.obstacle_drop(90, 40, side=8, centre=(35.0, 20.0), r_drop=7.0, drop_centre=(16.0, 20.0))
    else:
        wl = W.cocurrent("couette", nx=40, ny=42, a=10.0)
    wl.tau = 1.0
    return wl


@pytest.mark.parametrize("kind", ["walls", "periodic", "open", "couette"])
@pytest.mark.parametrize("tile", TILES[:4])
def test_fp64_against_oracle(oracle_mod, lbm_mod, kind, tile):
    wl = _case(kind)
    o = oracle_mod.Oracle(wl.nx, wl.ny, wl.flags)
    g = lbm_mod.lattice_from_workload(wl, lbm_mod.F64)
    g.set_tile(*tile)
    o.set_geometry(wl.solid)
    o.set_params(wl.G_c, wl.G_ads, wl.tau)
    o.set_body_accel(*wl.accel)
    if any(wl.wall_velocity):
        o.set_wall_velocity(*wl.wall_velocity)
    if wl.inlet_u is not None:
        o.set_inlet_velocity(wl.inlet_u[0], wl.inlet_u[1])
    o.init_fields(wl.rho1, wl.rho2)
    for q in (o, g):
        q.step(41)
    a, b = g.get_populations(), o.get_populations()
    assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))


@pytest.mark.parametrize("storage,flags", [(0, 0), (1, 0), (2, 0), (2, 1024), (3, 0), (3, 1024)])
@pytest.mark.parametrize("kind", ["walls", "periodic", "open", "couette"])
def test_tiles_equal_bricks(lbm_mod, kind, storage, flags):
    wl = _case(kind)
    ref = lbm_mod.lattice_from_workload(wl, storage, flags)  # bricks
    for q in (3, 8):
        ref.step(q)
    want = ref.get_populations()
    for tile in TILES:
        if storage == 0 and tile[0] == 256 and tile[2] & 8:
            continue  # FP64 fuses in 64 or 128 threads
        g = lbm_mod.lattice_from_workload(wl, storage, flags)
        g.set_tile(*tile)
        g.set_diag_interval(4)  # steps 0, 4, 8 in the diagnostic passes
        for q in (3, 8):
            g.step(q)
        assert np.array_equal(g.get_populations(), want), tile
