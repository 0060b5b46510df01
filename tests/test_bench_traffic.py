"""The benchmark quotes counter bytes only for the sources and the tile they were
taken with: a changed rule of tiles, launch or kernel drops them, and so does a tile
set by hand."""
import json
import os
import shutil

import pytest

import bench


@pytest.fixture
def record(tmp_path, monkeypatch):
    """A copy of the sources with counter bytes recorded for it."""
    csrc = tmp_path / "paper_2505_22256_amd" / "csrc"
    shutil.copytree(os.path.join(bench.ROOT, "paper_2505_22256_amd", "csrc"), csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    f = tmp_path / "traffic.json"
    f.write_text(json.dumps({"kernel_hash": bench.kernel_source_hash(),
                             "f32": {"tile": bench.BY_LIBRARY, "bytes_per_launch": 5}}))
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(f))
    return csrc


def test_bytes_belong_to_the_tile(record):
    assert bench.measured_traffic("f32", bench.BY_LIBRARY) == 5
    assert bench.measured_traffic("f32", {"block": 128, "seg_rows": 24, "sched": 10}) is None
    assert bench.measured_traffic("f16", bench.BY_LIBRARY) is None


@pytest.mark.parametrize("name", ["lbm_plan.hpp", "lbm_api.hip", "lbm_launch_impl.hpp", "lbm_kernels.hpp"])
def test_a_changed_source_drops_them(record, name):
    with open(record / name, "a") as f:
        f.write("// changed\n")
    assert bench.measured_traffic("f32", bench.BY_LIBRARY) is None
