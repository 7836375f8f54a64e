"""The files whose hash keys the bench's committed counter records: everything
of the library's that the kernels' compilation reads, and the dispatch."""
import os
import re
import subprocess

import pytest

import bench
from paper_1108_0486_amd import build as B


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not found")
def test_records_are_keyed_to_every_source(tmp_path):
    listed = {os.path.basename(p) for p in bench.KERNEL_SOURCES}
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
    out = tmp_path / "xg_kernels.i"
    subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-E", "-I", B.INCLUDE, "-I", B.CSRC,
                    os.path.join(B.CSRC, "xg_kernels.hip"), "-o", str(out)], check=True, capture_output=True)
    read = {os.path.basename(m) for m in re.findall(r'^# \d+ "([^"]*/csrc/[^"]*)"', out.read_text(), re.M)}
    assert "xg_kernels.hip" in read and "xg_split.h" in read
    assert read <= listed
    assert {"xg_api.cpp", "xg_shape.h"} <= listed
