"""The host rules of launches whose rows are cut into parts, and the jump
polynomials written for them at build time, under the sanitizers (CPU)."""
import os
import shutil
import subprocess

import pytest

from paper_1108_0486_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(not os.path.exists(B.HIPCC) or shutil.which("g++") is None, reason="hipcc or g++ not found")
def test_split_plans_and_tables(tmp_path):
    B.split_tables(str(tmp_path))
    exe = str(tmp_path / "split_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", B.INCLUDE, "-I", B.CSRC, "-I", str(tmp_path),
                    os.path.join(HERE, "sanitize", "split_driver.cpp"), os.path.join(B.CSRC, "xg_jump.cpp"),
                    "-o", exe], check=True)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and p.stdout.rstrip().endswith("OK"), p.stdout + p.stderr
