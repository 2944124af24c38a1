"""Traffic summaries are dropped when the sources of their kernel change."""
import os
import shutil

import pytest

from paper_1002_1202_amd import rocprof_summary


@pytest.mark.parametrize("name", ["cheb_step", "cheb_mx"])
@pytest.mark.parametrize("source", ["spmm.hip", "spmm.h", "kernels.h", "geometry.h"])
def test_digest_covers_sources(tmp_path, monkeypatch, name, source):
    """The block order and the row groups of a launch (geometry.h) set its traffic too."""
    shutil.copytree(os.path.join(rocprof_summary.HERE, "csrc"), tmp_path / "csrc")
    monkeypatch.setattr(rocprof_summary, "HERE", str(tmp_path))
    summary = tmp_path / "traffic.md"
    summary.write_text(f"- kernel: {name}\n- traffic_bytes_per_dispatch: 1.5e+08\n"
                       f"- source_digest: {rocprof_summary.source_digest(name)}\n")
    assert rocprof_summary.read_traffic(str(summary), name) == 1.5e8
    with open(tmp_path / "csrc" / source, "a") as f:
        f.write("// changed\n")
    assert rocprof_summary.read_traffic(str(summary), name) is None
