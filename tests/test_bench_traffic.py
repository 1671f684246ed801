"""The recorded HBM traffic that bench.py reports counts only for the sources
that it was measured on: a change to any file the kernel is made of voids it."""
import os
import shutil

import pytest

import bench

CSRC = os.path.join(bench.ROOT, "paper_2412_05082_amd", "csrc")
ROW = "| variant 1 | `kernel` | 1 | 1.0 | 1.0 | 1 (x1.00) | 4321 |\n"


@pytest.fixture
def recorded(tmp_path, monkeypatch):
    """A copy of the sources, with a record taken on it."""
    copy = tmp_path / "csrc"
    shutil.copytree(CSRC, copy)
    monkeypatch.setattr(bench, "KERNEL_SRCS", [str(copy / os.path.basename(p)) for p in bench.KERNEL_SRCS])
    monkeypatch.setattr(bench, "COUNTERS", str(tmp_path / "counters.md"))
    (tmp_path / "counters.md").write_text(f"kernel source sha256: {bench.kernel_digest()}\n\n{ROW}")
    return copy


def test_record_of_these_sources_counts(recorded):
    assert bench.measured_traffic(1) == 4321
    assert bench.measured_traffic(0) is None


@pytest.mark.parametrize("name", ["smooth2d_impl.h", "tile2d.h", "refband.h", "tiles.h", "gen_refcoef.cpp"])
def test_change_of_any_source_voids_the_record(recorded, name):
    with open(recorded / name, "a") as f:
        f.write("\n")
    assert bench.measured_traffic(1) is None
