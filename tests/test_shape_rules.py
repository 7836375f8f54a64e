"""The host rules that pick a plain launch's kernel by its sizes, compiled with
a host compiler under the sanitizers (CPU; 256 compute units)."""
import os
import shutil
import subprocess

import pytest

from paper_1108_0486_amd import build as B
from paper_1108_0486_amd import xg

from split_cases import EXPONENTS, LONGEST

HERE = os.path.dirname(os.path.abspath(__file__))
U32, F32, NORMAL, MOMENTS, U64, F64 = xg.XG_U32, xg.XG_F32, xg.XG_NORMAL, 3, 4, 5

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("shape") / "shape_driver")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", B.INCLUDE, "-I", B.CSRC, os.path.join(HERE, "sanitize", "shape_driver.cpp"), "-o", exe],
                   check=True)

    def ask(*cases):
        text = "\n".join(" ".join(str(v) for v in c) for c in cases)
        p = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=60)
        assert p.returncode == 0, p.stderr
        return [tuple(int(v) for v in line.split()) for line in p.stdout.splitlines()]
    return ask


# (family, kind, count, n, address, cached): sizes at which the other choice
# was measured slower, on either side of each line.
STORES = [
    # Short launches keep non-temporal stores, on whole lines ...
    (0, U32, 2048, 1 << 11, 0, 0), (0, U32, 2048, 1 << 12, 0, 0), (0, F32, 4096, 1 << 10, 0, 0),
    (1, U32, 2048, 1 << 13, 0, 0), (1, U32, 4096, 1 << 11, 0, 0), (2, U64, 2048, 1 << 11, 0, 0),
    # ... and off them.
    (0, U32, 4096, 1000, 0, 0), (0, U32, 4096, 1024, 4, 0), (1, F32, 4096, 1000, 0, 0), (2, U64, 3000, 1000, 0, 0),
    (0, NORMAL, 4096, 1000, 0, 0), (0, NORMAL, 2048, 5001, 0, 0), (1, NORMAL, 6000, 1000, 0, 0),
    (2, NORMAL, 6000, 1000, 0, 0),
    # Launches of many more streams than run at once.
    (0, U32, 20000, 1 << 13, 0, 0), (0, U32, 65536, 1 << 11, 0, 0), (1, U32, 20000, 1 << 13, 0, 0),
    (2, F64, 20000, 1 << 13, 0, 0), (0, U32, 20000, 1 << 11, 0, 1),
    # FP32 of the 32-bit r = 64 member with one wavefront per SIMD.
    (1, F32, 2048, 1 << 19, 0, 0), (1, F32, 2048, 1 << 15, 0, 1), (1, F32, 4096, 1 << 16, 0, 1),
    (1, U32, 2048, 1 << 19, 0, 1),
    # Long ones gain from cached stores.
    (0, U32, 2048, 1 << 13, 0, 1), (0, U32, 4096, 1 << 18, 0, 1), (0, U32, 12000, 1 << 12, 0, 1),
    (2, F64, 1300, 1 << 17, 0, 1), (2, U64, 1024, 1 << 17, 0, 0), (2, U64, 2048, 1 << 12, 0, 1),
    (2, U64, 2048, 1 << 13, 0, 1), (2, U64, 4096, 1 << 16, 0, 1),
    (0, U32, 4096, 65537, 0, 1), (0, U32, 1024, 100003, 0, 1), (0, NORMAL, 1024, 100003, 0, 1),
    (0, U32, 2300, 2500, 0, 1), (1, NORMAL, 3001, 65537, 0, 1), (2, NORMAL, 6000, 5001, 0, 1),
    # One wavefront per SIMD of Section 2's member, and normals on whole lines, never.
    (0, U32, 1024, 1 << 20, 0, 0), (0, NORMAL, 4096, 1 << 18, 0, 0), (1, NORMAL, 4096, 1 << 18, 0, 0),
    (0, MOMENTS, 4096, 65537, 0, 0),
]


def test_stores(rules):
    got = rules(*[("stores", *c[:5]) for c in STORES])
    assert [(c, g) for c, (g,) in zip(STORES, got) if g != c[5]] == []


@pytest.mark.parametrize("family,kind", [(0, U32), (0, NORMAL), (1, U32), (1, NORMAL), (2, U64), (2, NORMAL)])
def test_parts_of_every_exponent(rules, family, kind):
    got = rules(*[("split", family, kind, 1, n) for n in EXPONENTS.values()])
    assert got == [(129, e) for e in EXPONENTS]


@pytest.mark.parametrize("family,kind", [(0, U32), (0, NORMAL), (1, U32), (1, NORMAL), (2, U64), (2, NORMAL)])
def test_longest_rows_that_are_cut(rules, family, kind):
    per = 1 if family == 0 else 2
    got = rules(*[("split", family, kind, per * waves, n) for waves, n, _, _ in LONGEST])
    assert got == [(parts, e) for _, _, parts, e in LONGEST]
