"""Contact angles where the device's region words and link lists have their
edges: rows shorter than, as long as and longer than a 64-node word, node
counts that leave a ragged last word, many pockets and satellites, lattices
over several workgroups, and runs of a batch at unaligned offsets.  Against
the oracle on the same densities (no steps), FP64: the two differ by rounding
in the fit alone, 1e-9 degrees."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu


def _cap(shape, seed, r):
    """A cap of radius r on the wall plane 0 (last axis-0 plane solid too) with
    random pockets and satellites away from its rim."""
    rng = np.random.default_rng(seed)
    ax = np.meshgrid(*[np.arange(n, dtype=float) for n in shape], indexing="ij")
    h, rest = ax[0], ax[1:]
    d = np.sqrt((h - 0.5) ** 2 + sum((a - n / 2.0) ** 2 for a, n in zip(rest, shape[1:])))
    s = np.tanh((r - d) / 1.5)
    flip = (np.abs(d - r) > 3.0) & (rng.random(shape) < 0.15)
    s = np.where(flip, -s, s) * (1.0 - 0.01 * rng.random(shape))
    solid = np.zeros(shape, np.uint8)
    solid[0] = solid[-1] = 1
    rho = [np.where(solid, 0.0, 0.52 + sign * 0.43 * s) for sign in (1.0, -1.0)]
    return solid, rho


def _workload(nx, ny, seed, r):
    solid, rho = _cap((ny, nx), seed, r)
    return W.Workload("cap", nx, ny, W.PERIODIC_X, solid, rho[0], rho[1], wall_kind=W.WALL_FLAT, wall=(0.5, 0.0, 0.0))


@pytest.mark.parametrize("nx,ny,r", [(31, 23, 9.0), (63, 40, 15.0), (64, 41, 16.0), (65, 37, 16.0), (130, 67, 31.0),
                                     (517, 260, 110.0)])
def test_angle_with_pockets(oracle_mod, lbm_mod, nx, ny, r):
    wl = _workload(nx, ny, nx, r)
    o = oracle_mod.Oracle(nx, ny, wl.flags)
    o.set_geometry(wl.solid)
    o.set_params(wl.G_c, wl.G_ads, wl.tau)
    o.init_fields(wl.rho1, wl.rho2)
    g = lbm_mod.lattice_from_workload(wl, lbm_mod.F64)
    assert abs(g.contact_angle(0, wl.wall) - o.contact_angle(0, wl.wall)) < 1e-9


def test_batch_angles_are_those_of_single_runs(lbm_mod):
    runs = [_workload(nx, ny, nx + ny, 0.24 * nx) for nx, ny in ((37, 29), (64, 33), (131, 64), (66, 47), (65, 41))]
    b = lbm_mod.Batch(runs, lbm_mod.F64)
    got = b.contact_angles()
    for th, wl in zip(got, runs):
        assert th == lbm_mod.lattice_from_workload(wl, lbm_mod.F64).contact_angle(0, wl.wall)


@pytest.mark.parametrize("nx,ny,nz,r", [(21, 22, 17, 8.0), (33, 31, 20, 11.0), (64, 66, 24, 14.0)])
def test_angle_with_pockets_3d(oracle_mod, lbm_mod, nx, ny, nz, r):
    solid, rho = _cap((nz, ny, nx), nx, r)
    lats = [oracle_mod.Oracle3D(nx, ny, nz, 3), lbm_mod.Lattice3D(nx, ny, nz, lbm_mod.F64, 3)]
    for q in lats:
        q.set_geometry(solid)
        q.set_params(0.9, 0.0, 1.0)
        q.init_fields(rho[0], rho[1])
    to, tg = (q.contact_angle(0, (0.5, 0.0, 0.0, 0.0)) for q in lats)
    assert abs(tg - to) < 1e-9


# labels are joined in bands of 4096 nodes: rows longer than a band, bands that
# end with a row and inside one, one node into a second band
@pytest.mark.parametrize("nx,ny,r", [(5000, 23, 9.0), (4096, 21, 9.0), (128, 97, 30.0), (100, 90, 28.0), (241, 17, 9.0)])
def test_angle_over_label_bands(oracle_mod, lbm_mod, nx, ny, r):
    wl = _workload(nx, ny, nx + 1, r)
    o = oracle_mod.Oracle(nx, ny, wl.flags)
    o.set_geometry(wl.solid)
    o.set_params(wl.G_c, wl.G_ads, wl.tau)
    o.init_fields(wl.rho1, wl.rho2)
    g = lbm_mod.lattice_from_workload(wl, lbm_mod.F64)
    assert abs(g.contact_angle(0, wl.wall) - o.contact_angle(0, wl.wall)) < 1e-9


@pytest.mark.parametrize("nx,ny,nz", [(64, 64, 20), (71, 70, 19)])  # a plane is a band; a plane is longer
def test_angle_over_label_bands_3d(oracle_mod, lbm_mod, nx, ny, nz):
    solid, rho = _cap((nz, ny, nx), nx + 1, 11.0)
    lats = [oracle_mod.Oracle3D(nx, ny, nz, 3), lbm_mod.Lattice3D(nx, ny, nz, lbm_mod.F64, 3)]
    for q in lats:
        q.set_geometry(solid)
        q.set_params(0.9, 0.0, 1.0)
        q.init_fields(rho[0], rho[1])
    to, tg = (q.contact_angle(0, (0.5, 0.0, 0.0, 0.0)) for q in lats)
    assert abs(tg - to) < 1e-9
