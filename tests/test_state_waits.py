"""Where the compiled word kernels of the r = 64 members wait for their state,
read from the AMD assembly of this repository's own kernel source built for
gfx950 (no GPU needed).

One counter serves a wavefront's loads and stores in order.  A state word whose
first use comes after the loop of stores was waited for there, which is a wait
for every store of the row; the kernels wait for the whole state in front of
the loop instead."""
import os
import re
import subprocess

import pytest

from paper_1108_0486_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not found")


def test_no_load_is_waited_for_after_a_store(tmp_path):
    out = tmp_path / "xg_family.s"
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([B.HIPCC, *flags, "--cuda-device-only", "-S", "-I", B.INCLUDE, "-I", B.CSRC,
                    os.path.join(B.CSRC, "xg_family.hip"), "-o", str(out)], check=True, capture_output=True)
    kernels = re.findall(r"^(_ZN2xg12_GLOBAL__N_114k_fam_generate\S*):\s*;(.*?)^\.Lfunc_end", out.read_text(),
                         re.S | re.M)
    assert len(kernels) >= 32
    for name, body in kernels:
        ops = [line.split(";")[0].strip() for line in body.split("\n")]
        first = next(i for i, op in enumerate(ops) if op.startswith("global_store"))
        late = [op for op in ops[first:] if op.startswith("s_waitcnt") and "vmcnt" in op]
        assert not late, (name, late)
