"""The guard on the recorded HBM traffic of the dominant GEMM: bench.py
reports the figure only while every file that defines what the kernel reads
and writes is the one it was measured with."""
import json
import os
import shutil

import pytest

import bench
from paper_2608_07974_amd.profile_summary import GEMM_SOURCES, sources_sha256


@pytest.mark.parametrize("changed", [None] + [os.path.basename(p) for p in GEMM_SOURCES])
def test_traffic_is_reported_only_for_the_measured_sources(tmp_path, changed):
    src = [shutil.copy(p, tmp_path) for p in GEMM_SOURCES]
    rec = tmp_path / "record.json"
    rec.write_text(json.dumps({"kernels": [dict(kernel="k", workload="w", source_sha256=sources_sha256(src),
                                                hbm_bytes_per_launch=7)]}))
    if changed:
        with open(tmp_path / changed, "a") as f:
            f.write("\n// changed\n")
    assert bench.measured_traffic("k", "w", rec, src) == (None if changed else 7)
    assert bench.measured_traffic("other", "w", rec, src) is None


def test_the_guard_covers_the_kernel_and_its_epilogue():
    assert {os.path.basename(p) for p in GEMM_SOURCES} >= {"gemm_tiles.h", "gemm_epilogue.h", "gemm.hip"}
    assert all(os.path.exists(p) for p in GEMM_SOURCES)
