"""One stream's row cut into parts of every length there is (2^12 to 2^20
values, 129 parts, and the longest row that is cut, 256 parts), against the
same call in an explicit launch shape, which is never cut, and against the
stream skipped to a part's start."""
import pytest

from gpu_helpers import needs_gpu
from split_cases import EXPONENTS

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd.streams import XorgensStreams  # noqa: E402


def _bits(t):
    return t.view(torch.int64 if t.element_size() == 8 else torch.int32)


def _check(family, call, n, parts, exp):
    a, b, c = (XorgensStreams(1, seed=31, family=family) for _ in range(3))
    b.set_plain_tune(1, 8, 1)
    x = getattr(a, call)(n).view(-1)
    y = getattr(b, call)(n).view(-1)
    assert torch.equal(_bits(x), _bits(y))
    assert torch.equal(a.state, b.state)
    del y
    at = 0
    for k in (1, 2, 64, 96, 127, parts - 1):  # odd and even multiples of the part
        c.skip((k << exp) - 64 - at)
        z = getattr(c, call)(320).view(-1)
        assert torch.equal(_bits(z), _bits(x[(k << exp) - 64:(k << exp) + 256])), k
        at = (k << exp) + 256


@pytest.mark.parametrize("exp", list(EXPONENTS))
@pytest.mark.parametrize("family,call", [(0, "u32"), (0, "normal"), (1, "f32"), (1, "normal"), (2, "u64"),
                                         (2, "normal_f64")])
def test_parts_of_every_exponent(family, call, exp):
    _check(family, call, EXPONENTS[exp], 129, exp)


@pytest.mark.parametrize("family,call", [(0, "f32"), (1, "u32")])
def test_the_longest_row(family, call):
    _check(family, call, (1 << 28) + 255, 256, 20)


@pytest.mark.parametrize("family,count", [(0, 2), (1, 3), (2, 4)])
@pytest.mark.parametrize("exp", [12, 15, 18])
def test_bulk_fill(family, count, exp):
    """Several streams in the bulk-fill layout; the parts' tails lie behind it."""
    a, b = XorgensStreams(count, seed=8, family=family), XorgensStreams(count, seed=8, family=family)
    b.set_plain_tune(1, 8, 1)
    call = "fill_f64" if family == 2 else "fill_u32"
    x, y = getattr(a, call)(EXPONENTS[exp]), getattr(b, call)(EXPONENTS[exp])
    assert torch.equal(_bits(x), _bits(y)) and torch.equal(a.state, b.state)
