"""Launches of few streams, whose rows are cut into parts that start from
jumped states (xg_split.h), against the oracle, and against the same call in
an explicit launch shape, which is never split."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu, ulp32_error
from oracle import oracle as O

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd import xg  # noqa: E402
from paper_1108_0486_amd.streams import XorgensStreams, as_u32  # noqa: E402

PART = 1 << 11   # the shortest part
FAMILIES = [xg.XG_FAMILY_R128_W32, xg.XG_FAMILY_R64_W32, xg.XG_FAMILY_R64_W64]


def _calls(family):
    if family == xg.XG_FAMILY_R64_W64:
        return ["u64", "f64", "fill_u64", "fill_f64", "normal_f64"]
    return ["u32", "f32", "fill_u32", "fill_f32", "normal"]


@pytest.mark.parametrize("family", FAMILIES)
@pytest.mark.parametrize("count,n", [
    (1, 3000),                       # too short to be split
    (1, 17 * PART + 255),            # the rest stays with the last part
    (1, 17 * PART + 256),            # the shortest last part
    (1, 17 * PART + 257),
    (1, 1 << 15),
    (1, 256 * PART + 255),           # the most parts of the shortest length
    (1, 256 * PART + 256),           # the next length
    (3, 100_003),
    (2, 1 << 20),
    (101, 40_001),
    (512, 140_001),                  # the most streams (R128)
    (1023, 140_001),                 # the most pairs of streams, one stream alone
])
def test_split_equals_unsplit(family, count, n):
    """Every output bit and end state of every kind of call, from a position
    that is not a whole number of steps, on a part of the streams."""
    a = XorgensStreams(count + 3, seed=42, family=family)
    b = XorgensStreams(count + 3, seed=42, family=family)
    b.set_plain_tune(1, 8, 1)
    for gs in (a, b):
        getattr(gs, _calls(family)[0])(133)
    for call in _calls(family):
        x, y = getattr(a, call)(n, first=2, count=count), getattr(b, call)(n, first=2, count=count)
        bits = torch.int64 if x.element_size() == 8 else torch.int32
        assert torch.equal(x.view(bits), y.view(bits)), call
        assert torch.equal(a.state, b.state), call


def test_split_against_oracle():
    gs, ref = XorgensStreams(2, seed=7), O.OracleStreams(7, 2)
    n = 5 * 8192 + 777
    assert (as_u32(gs.u32(n)) == ref.u32(n)).all()
    assert (gs.f32(n).cpu().numpy() == ref.f32(n)).all()
    z, want = gs.normal(n).cpu().numpy(), ref.normal(n)
    assert ulp32_error(z, want).max() <= 4.0
    got = as_u32(gs.fill_u32(n))
    want = ref.u32(n)
    assert (got[xg.fill_index(2, n)] == want).all()
    ring, weyl, pos = gs.host_state()
    assert (ring == ref.ring).all() and (weyl == ref.weyl).all() and (pos == ref.pos).all()


def test_split_stays_inside_its_output():
    """Rows at an odd offset in a larger buffer: nothing outside is touched."""
    gs = XorgensStreams(3, seed=5)
    buf = torch.full((3 * 50_001 + 2000,), -7, dtype=torch.int32, device="cuda")
    for call in ("u32", "fill_u32"):
        buf.fill_(-7)
        getattr(gs, call)(50_001, out=buf[1001:1001 + 3 * 50_001])
        assert (buf[:1001] == -7).all() and (buf[1001 + 3 * 50_001:] == -7).all(), call


def test_split_in_a_graph():
    a, b = XorgensStreams(4, seed=9), XorgensStreams(4, seed=9)
    out = torch.empty((4, 70_001), dtype=torch.float32, device="cuda")
    a.normal(70_001, out=out)
    b.normal(70_001)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        a.normal(70_001, out=out)
    for replay in range(3):
        g.replay()
        torch.cuda.synchronize()
        want = b.normal(70_001)
        assert torch.equal(out, want) and torch.equal(a.state, b.state), replay


@pytest.mark.parametrize("family,count", [(0, 512), (0, 400), (1, 1024), (1, 901), (2, 1023)])
def test_half_of_the_simds(family, count):
    """As many streams as are ever cut, in two parts; the second one longer."""
    test_split_equals_unsplit(family, count, (1 << 18) + 133)
