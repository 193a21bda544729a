"""Traffic figures of the committed profiles count only while every source of their
kernel is the one they were taken on, headers included."""
import json
import os
import shutil

import pytest

import bench


@pytest.mark.parametrize("source,header", [
    ("cdd_block.hip", "cdd_mfma.h"), ("cdd_block.hip", "cdd_fft.h"),
    ("cdd_large.hip", "cdd_fullband.h"), ("cdd_large.hip", "cdd_internal.h")])
def test_a_changed_header_outdates_the_figures(tmp_path, monkeypatch, source, header):
    csrc = tmp_path / "csrc"
    shutil.copytree(bench.CSRC, csrc)
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "CSRC", str(csrc))
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    files = bench.kernel_sources(source)
    assert files[0] == source and header in files
    rec = dict(sources=files, source_digest=bench.source_digest(files), bytes_per_launch=7.0)
    with open(os.path.join(tmp_path, "profiles", "traffic.json"), "w") as fh:
        json.dump(dict(kernel=dict(load=rec)), fh)
    assert bench.measured_traffic("kernel", "load") == 7.0
    with open(csrc / header, "a") as fh:
        fh.write("// changed\n")
    assert bench.measured_traffic("kernel", "load") is None
