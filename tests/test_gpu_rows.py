"""Stream-major rows through the kernels with cached stores (rows that start
inside a cache line, two wavefronts or more per SIMD) against the same call in
an explicit launch shape, which never takes them, and the oracle."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu
from oracle import oracle as O

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd.streams import XorgensStreams, as_u32  # noqa: E402


@pytest.mark.parametrize("family,call", [(0, "u32"), (0, "f32"), (0, "normal"), (1, "u32"), (1, "f32"), (1, "normal"),
                                         (2, "u64"), (2, "f64"), (2, "normal_f64")])
@pytest.mark.parametrize("count", [1, 3, 700, 1027, 2049])
def test_rows_equal_explicit_shape(family, call, count):
    a, b = XorgensStreams(count, seed=4, family=family), XorgensStreams(count, seed=4, family=family)
    b.set_plain_tune(4, 4, 1)
    wide = family == 2
    dtype = (torch.float64 if wide else torch.float32) if call[0] in "fn" else (torch.int64 if wide else torch.int32)
    bits = torch.int64 if wide else torch.int32
    for n in (1, 63, 64, 65, 512, 513, 1024, 1056, 12000, 12032):   # 512, 1024, 1056, 12032: whole lines
        buf = torch.zeros(count * n + 9, dtype=dtype, device="cuda")
        for at in (0, 5):
            buf.zero_()
            getattr(a, call)(n, out=buf[at:at + count * n])
            want = getattr(b, call)(n)
            assert torch.equal(buf[at:at + count * n].view(bits), want.reshape(-1).view(bits)), (n, at)
            assert int(buf[:at].count_nonzero()) == 0 and int(buf[at + count * n:].count_nonzero()) == 0, (n, at)
            assert torch.equal(a.state, b.state), (n, at)


def test_rows_against_oracle():
    S, n = 2100, 4099   # over 32 MB, odd
    gs, ref = XorgensStreams(S, seed=8), O.OracleStreams(8, S)
    assert (as_u32(gs.u32(n)) == ref.u32(n)).all()
    assert (gs.f32(n).cpu().numpy() == ref.f32(n)).all()
    assert (as_u32(gs.u32(1024)) == ref.u32(1024)).all()
    ring, weyl, pos = gs.host_state()
    assert (ring == ref.ring).all() and (weyl == ref.weyl).all() and (pos == np.uint64(2 * n + 1024)).all()
