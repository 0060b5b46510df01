"""Batches around 64 runs (the owner of a work item is found 64 runs at a time)
and their step counters (one word per buffer side, advanced by the steps
themselves), which stochastic rounding makes visible: every run equal to the
same run alone, eager and replayed from a graph of an odd number of steps, with
two fused steps and one."""
import numpy as np
import pytest

from paper_2505_22256_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nruns", [1, 2, 63, 64, 65, 131])
@pytest.mark.parametrize("storage,sched,graph", [(2, 0, 3), (2, 8, 0), (3, 8, 5), (1, 0, 0)])
def test_every_run_equals_itself_alone(lbm_mod, nruns, storage, sched, graph):
    runs = [W.random_small(r, 14 + r % 23, 12 + (7 * r) % 19, 3, n_blobs=1) for r in range(nruns)]
    b = lbm_mod.Batch(runs, storage)
    b.set_sched(sched)
    b.set_tile(64, 8)
    if graph:
        b.use_graph(True, graph)
    for n in (7, 1, 12):
        b.step(n)
    for r in sorted({0, nruns // 2, nruns - 1, min(63, nruns - 1), min(64, nruns - 1)}):
        g = lbm_mod.lattice_from_workload(runs[r], storage)
        g.step(20)
        for x, y in zip(b.get_fields(r), g.get_fields()):
            assert np.array_equal(x, y), r
