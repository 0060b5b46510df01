"""Diagnostics recorded inside two fused steps, by the first of the pair and by the
second, with and without boundary code.  Populations equal those of one step per
launch (bitwise).  The record equals lbm_reduce of a single-step lattice at the
record's time: maxima, minima and the count exactly (the same arithmetic per
node), the sums to the rounding of their order, 1e-12 in FP64 and 1e-5 in FP32
and 16-bit storage (FP32 partial sums over at most 64 rows and a workgroup: 2^-24
times a few hundred terms), of the sum of the magnitudes.  FP64 against the
oracle too: 1e-12 of the masses and densities (the library's bound for FP64), and
velocities, quotients of momenta that are sums of 18 such populations by a density
of at least 0.9, to 1e-11."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu

TILES = [(64, 8, 8), (64, 24, 10), (128, 16, 10), (128, 0, 8), (256, 16, 10)]


def _case(kind):
    if kind == "open":
        wl = W.obstacle_drop(90, 40, side=8, centre=(35.0, 20.0), r_drop=7.0, drop_centre=(16.0, 20.0))
    elif kind == "obstacle":
        wl = W.obstacle_drop()
    elif kind == "couette":
        wl = W.cocurrent("couette", nx=140, ny=42, a=10.0)
    else:
        wl = W.random_small(5, 175, 41, 1, n_blobs=9, walls=True)
    wl.tau = 0.9
    return wl


def _oracle(oracle_mod, wl):
    o = oracle_mod.Oracle(wl.nx, wl.ny, wl.flags)
    o.set_geometry(wl.solid)
    o.set_params(wl.G_c, wl.G_ads, wl.tau)
    o.set_body_accel(*wl.accel)
    if any(wl.wall_velocity):
        o.set_wall_velocity(*wl.wall_velocity)
    if wl.inlet_u is not None:
        o.set_inlet_velocity(wl.inlet_u[0], wl.inlet_u[1])
    o.init_fields(wl.rho1, wl.rho2)
    return o


# records every 3 steps in calls of 5 and 2: boundaries on, the first step runs
# alone and 3 is the first of (3, 4), 6 the second of (5, 6); closed, 3 is the
# second of (2, 3) and 6 runs alone; in calls of 4 and 4, 6 is the first of (6, 7)
@pytest.mark.parametrize("calls", [(5, 2), (4, 4)])
@pytest.mark.parametrize("storage", [0, 1, 2, 3])
@pytest.mark.parametrize("kind", ["open", "obstacle", "couette", "walls"])
def test_records_of_fused_steps(oracle_mod, lbm_mod, kind, storage, calls):
    wl = _case(kind)
    ref = lbm_mod.lattice_from_workload(wl, storage)
    ref.set_tile(256, 16, 0)
    want, o = {}, _oracle(oracle_mod, wl) if storage == 0 else None
    for t in range(0, sum(calls), 3):
        n = t - ref.time
        ref.step(n)
        want[t] = ref.reduce(), None
        if o:
            o.step(n)
            want[t] = want[t][0], o.reduce()
    ref.step(sum(calls) - ref.time)
    pops = ref.get_populations()
    tol = 1e-12 if storage == 0 else 1e-5
    for tile in TILES:
        if storage == 0 and tile[0] == 256:
            continue  # FP64 fuses in 64 or 128 threads
        g = lbm_mod.lattice_from_workload(wl, storage)
        g.set_tile(*tile)
        g.set_diag_interval(3)
        for n in calls:
            g.step(n)
            d, t = g.get_diag()
            r, exact = want[t]
            assert t == (g.time - 1) // 3 * 3
            assert np.array_equal(d[4:], r[4:]), (tile, t)
            mass = r[0] + r[1]
            assert np.all(np.abs(d[:2] - r[:2]) <= tol * np.abs(r[:2])), (tile, t)
            assert np.all(np.abs(d[2:4] - r[2:4]) <= tol * mass * r[4]), (tile, t)
            if exact is not None:
                assert np.all(np.abs(d[:2] - exact[:2]) <= 1e-12 * exact[:2]), (tile, t)
                assert np.all(np.abs(d[2:4] - exact[2:4]) <= 1e-11 * mass), (tile, t)
                assert abs(d[4] - exact[4]) <= 1e-11, (tile, t)
                assert np.all(np.abs(d[5:7] - exact[5:7]) <= 1e-12 * exact[6]) and d[7] == 0, (tile, t)
        assert np.array_equal(g.get_populations(), pops), tile
