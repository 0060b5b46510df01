"""3-D steps at relaxation time 1, where the density pass leaves the momenta
and the collide pass pulls no populations.  FP64 against the oracle to 1e-12
(the library's bound for FP64); every storage and brick equal to the default
brick, on boxes narrower than a brick, ragged ones and closed ones; and the
default brick chooses its threads by size without changing the result."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu

BRICKS = [(32, 8, 4, 1), (32, 8, 4, 2), (32, 8, 4, 4), (32, 8, 8, 1), (32, 8, 8, 2), (64, 4, 4, 2)]


@pytest.mark.parametrize("nx,ny,nz,flags", [(14, 12, 10, 1 | 2 | 2048), (33, 9, 8, 1), (40, 17, 13, 0)])
def test_fp64_against_oracle(oracle_mod, lbm_mod, nx, ny, nz, flags):
    wl = W.random_small3d(nx, nx, ny, nz, flags)
    wl.tau = 1.0
    f = W.random_populations3d(3, wl, 0.1)
    o = oracle_mod.Oracle3D(nx, ny, nz, flags)
    g = lbm_mod.Lattice3D(nx, ny, nz, lbm_mod.F64, flags)
    for q in (o, g):
        q.set_geometry(wl.solid)
        q.set_params(wl.G_c, wl.G_ads, wl.tau)
        q.set_body_accel(wl.accel)
        q.set_populations(f)
        q.step(15)
    a, b = g.get_populations(), o.get_populations()
    assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))


@pytest.mark.parametrize("storage,rounding", [(0, 0), (1, 0), (2, 0), (2, 1024), (3, 0)])
@pytest.mark.parametrize("tau", [1.0, 0.8])
@pytest.mark.parametrize("nx,ny,nz", [(9, 30, 11), (70, 19, 21)])
def test_bricks_equal(lbm_mod, nx, ny, nz, tau, storage, rounding):
    wl = W.random_small3d(nx + nz, nx, ny, nz, 1 | 2048)
    wl.tau = tau
    want = None
    for brick in [None] + BRICKS:
        g = lbm_mod.lattice3d_from_workload(wl, storage, rounding)
        if brick:
            g.set_tile(*brick)
        g.step(7)
        got = g.get_populations()
        want = got if want is None else want
        assert np.array_equal(got, want), brick


def test_changing_the_relaxation_time(oracle_mod, lbm_mod):
    """The momenta belong to one step: steps at 1, at 0.7 and at 1 again."""
    wl = W.random_small3d(2, 20, 15, 12)
    o = oracle_mod.Oracle3D(20, 15, 12, wl.flags)
    g = lbm_mod.Lattice3D(20, 15, 12, lbm_mod.F64, wl.flags)
    for q in (o, g):
        q.set_geometry(wl.solid)
        q.set_params(wl.G_c, wl.G_ads, 1.0)
        q.init_fields(wl.rho1, wl.rho2)
        for tau in (1.0, 0.7, 1.0):
            q.set_params(wl.G_c, wl.G_ads, tau)
            q.step(3)
    a, b = g.get_populations(), o.get_populations()
    assert np.max(np.abs(a - b)) <= 1e-12 * np.max(np.abs(b))
