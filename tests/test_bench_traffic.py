"""bench.py reports a recorded traffic figure only beside the kernel, the sources and the refresh
period that it was recorded for."""
import json
import os
import shutil

import pytest

import bench

KERNEL = "k_cg_tile + k_refresh_tile"


@pytest.fixture
def root(tmp_path, monkeypatch):
    csrc = tmp_path / "paper_2604_02266_amd" / "csrc"
    csrc.mkdir(parents=True)
    (tmp_path / "profiles").mkdir()
    for name in bench.KERNEL_SRC:
        shutil.copy(os.path.join(bench.ROOT, "paper_2604_02266_amd", "csrc", name), csrc)
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    with open(tmp_path / "profiles" / "traffic_w.json", "w") as f:
        json.dump({"kernel": KERNEL, "kernel_source_sha": bench.kernel_source_sha(), "refresh_every": 10,
                   "traffic_bytes_per_launch": 123.0}, f)
    return tmp_path


def test_traffic_of_the_present_sources(root):
    assert bench.load_traffic("w", 10, KERNEL) == 123.0
    assert bench.load_traffic("other", 10, KERNEL) is None


def test_another_kernel_or_period(root):
    assert bench.load_traffic("w", 10, "k_cg_fused + k_refresh_u + k_refresh_c") is None
    assert bench.load_traffic("w", 0, KERNEL) is None


@pytest.mark.parametrize("name", ["kernels.hip", "cg_tile.hip", "device_util.h", "otfs_internal.h"])
def test_changed_sources(root, name):
    with open(root / "paper_2604_02266_amd" / "csrc" / name, "a") as f:
        f.write("\n")
    assert bench.load_traffic("w", 10, KERNEL) is None
