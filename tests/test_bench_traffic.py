"""The benchmark's profiled HBM traffic of the m = 32 upscaling kernel is reported
only while the kernel's code is the one that was profiled: its file and every
header of the package that it includes."""
import os
import shutil

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def tree(tmp_path, monkeypatch):
    shutil.copytree(os.path.join(ROOT, "paper_1607_00693_amd", "csrc"), tmp_path / "paper_1607_00693_amd" / "csrc")
    os.makedirs(tmp_path / "profiles")
    shutil.copy(os.path.join(ROOT, "profiles", "upscale_mesh32_hbm_traffic.md"), tmp_path / "profiles")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    return tmp_path


def test_profile_is_of_this_kernel():
    assert bench.profiled_traffic_per_pair() is not None


@pytest.mark.parametrize("name", ["upscale_rows.hip", "band_rows.h", "small_cell.h", "common.h"])
def test_a_changed_source_is_noticed(tree, name):
    assert bench.profiled_traffic_per_pair() is not None
    with open(tree / "paper_1607_00693_amd" / "csrc" / name, "a") as f:
        f.write("// changed\n")
    assert bench.profiled_traffic_per_pair() is None
