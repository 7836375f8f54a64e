"""When groups of different lengths of an r = 64 batch run alone in a wavefront:
the device's rule, compiled with a host compiler under the sanitizers (CPU)."""
import os
import shutil
import subprocess

import pytest

from paper_1108_0486_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))

# (64 bits, normals, requests a group, words of the largest group, mean words of
# the groups second on their SIMD, alone): tables at which the other choice was
# measured at least a tenth slower, or, for short ones, slower at all.
CASES = [
    # 2000 groups of nearly equal or uniform lengths up to 2^16 and 2^15: pairs.
    (1, 1, 1, 65536, 62900, 0), (0, 1, 1, 65536, 62900, 0), (1, 1, 1, 65536, 32000, 0), (0, 1, 1, 32768, 31400, 0),
    # Two requests each of 2^15 and 2^16.
    (1, 1, 2, 65536, 62900, 0), (0, 1, 2, 131072, 131072, 0), (1, 1, 2, 131072, 131072, 0),
    # Four of 2^15.
    (1, 1, 4, 131072, 131072, 0),
    # Short ones, or none second on a SIMD: alone.
    (0, 0, 1, 4000, 0, 1), (1, 0, 1, 4000, 0, 1), (0, 1, 1, 4000, 0, 1), (1, 1, 1, 4000, 0, 1),
    (0, 1, 4, 16384, 0, 1), (1, 1, 4, 16384, 0, 1), (0, 0, 4, 12000, 4800, 1), (1, 0, 4, 12000, 4800, 1),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_lone_groups_follow_what_they_save_and_cost(tmp_path):
    exe = str(tmp_path / "pairs_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", B.INCLUDE, "-I", B.CSRC, os.path.join(HERE, "sanitize", "pairs_driver.cpp"), "-o", exe],
                   check=True)
    text = "\n".join(" ".join(str(v) for v in c[:5]) for c in CASES)
    p = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stderr
    got = [int(v) for v in p.stdout.split()]
    assert [c for c, g in zip(CASES, got) if c[5] != g] == [] and len(got) == len(CASES)
