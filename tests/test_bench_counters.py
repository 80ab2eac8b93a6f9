"""bench.py's counter record: which sources, layout and shape it holds for (no GPU)."""

import json
import os
import shutil
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


@pytest.mark.parametrize("source", ["dslash.hip", "dslash_kernel.h", "dslash_f32.hip", "hisq_internal.h", "pack.hip"])
def test_counter_record_holds_for_its_kernel_sources_only(tmp_path, monkeypatch, source):
    """The committed bytes per launch are reported for the sources they were
    counted with, and no longer once one of them, the shape or the layout differs."""
    import bench
    csrc = os.path.join("paper_2111_10354_amd", "csrc")
    shutil.copytree(os.path.join(ROOT, csrc), tmp_path / csrc)
    shutil.copytree(os.path.join(ROOT, "profiles"), tmp_path / "profiles")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    dims = (96, 96, 96, 24)
    with open(tmp_path / "profiles" / "dslash_fp32_96x96x96x24.traffic.json") as f:
        rec = json.load(f)
    shape = rec["launch_shape"]
    assert bench.counter_traffic(dims, False, shape) == rec["traffic_bytes_per_launch"] / 1e9
    assert bench.counter_traffic(dims, True, shape) is None
    assert bench.counter_traffic(dims, False, [shape[0], shape[1] * 2, shape[2]]) is None
    with open(tmp_path / csrc / source, "a") as f:
        f.write("// changed\n")
    assert bench.counter_traffic(dims, False, shape) is None
