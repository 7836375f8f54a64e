"""Stored normals and moments of the 32-bit members with more than one wavefront
per SIMD (pairs gathered through LDS, two 128-normal blocks at a time) around
the edges of blocks and unrolled groups, against a launch of one stream at a
time (pairs gathered in the VALU) and the oracle."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu, ulp32_error
from oracle import oracle as O

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd.streams import XorgensStreams  # noqa: E402


@pytest.mark.parametrize("unroll", [0, 1, 2, 4, 8])
@pytest.mark.parametrize("family", [0, 1])
@pytest.mark.parametrize("n", [1, 127, 128, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2051, 4099])
def test_many_streams_equal_few(unroll, family, n):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    S = (4 if family == 0 else 8) * cus + 5
    many, few = XorgensStreams(S, seed=3, family=family), XorgensStreams(S, seed=3, family=family)
    if unroll:
        many.set_plain_tune(4, unroll, 1)
    buf = torch.full((S * n + 6,), 5.0, dtype=torch.float32, device="cuda")
    z = many.normal(n, out=buf[3:3 + S * n])
    assert (buf[:3] == 5.0).all() and (buf[3 + S * n:] == 5.0).all()
    z = buf[3:3 + S * n].view(S, n)
    rows = [0, 1, S // 2, S - 2, S - 1]
    for i in rows:
        assert torch.equal(few.normal(n, first=i, count=1)[0], z[i]), i
    st = few.state.numel() // S if family == 0 else 68
    for i in rows:
        assert torch.equal(few.state[i * st:(i + 1) * st], many.state[i * st:(i + 1) * st]), i
    m = many.moments(n).cpu().numpy().astype(np.float64)
    ref = O.OracleStreams(3, S, params=O.PAPER if family == 0 else O.R64)
    ref.normal(n)
    want = ref.normal(n)
    u = 2.0 ** -24
    assert (np.abs(m[:, 0] - want.sum(1)) <= 27 * u * np.abs(want).sum(1)).all()
    assert (np.abs(m[:, 1] - (want * want).sum(1)) <= 27 * u * (want * want).sum(1)).all()
    assert ulp32_error(many.normal(n)[rows].cpu().numpy(), ref.normal(n)[rows]).max() <= 4.0
