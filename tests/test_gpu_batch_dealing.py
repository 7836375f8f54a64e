"""Which batches' items are dealt to the wavefronts and which are taken from the
queue (its counter, word 0 of the workspace, then moves): by the cost of the
first item that is not some wavefront's first, however its requests share it;
and the values and end states either way, against plain launches."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd.batch import Batch  # noqa: E402
from paper_1108_0486_amd.streams import XorgensStreams  # noqa: E402

SHAPE = (1, 8, 1, 1)  # one wavefront per compute unit


def _run(family, lengths, groups):
    """A batch of `groups` streams with requests of these lengths each; the
    queue counter it leaves."""
    per = sum(lengths)
    reqs = []
    for s in range(groups):
        at = s * per
        for n in lengths:
            reqs.append((s, n, at, 0))
            at += n
    a, b = XorgensStreams(groups, seed=9, family=family), XorgensStreams(groups, seed=9, family=family)
    batch = Batch(a, reqs, groups * per)
    batch.out.zero_()
    batch.run(tune=SHAPE)
    want = (b.u64 if family == 2 else b.u32)(per)
    assert torch.equal(batch.out[:groups * per].view(groups, per), want)
    assert torch.equal(a.state, b.state) and batch.error_flag() == 0
    return int(batch.scratch[0].item())


def _groups(family):
    """More than every wavefront's first item (two groups each for r = 64)."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return (1 if family == 0 else 2) * cus + 41


@pytest.mark.parametrize("family", [0, 1, 2])
def test_a_short_first_request_does_not_hide_a_long_one(family):
    assert _run(family, (1, 70000), _groups(family)) > 0


@pytest.mark.parametrize("family", [0, 1, 2])
@pytest.mark.parametrize("tail", [1, 3, 63, 64, 65])
def test_a_long_first_request_is_counted_once(family, tail):
    """Costs just below the limits (2^16 words; 2^12 of the r = 64 members)."""
    assert _run(family, ((60000 if family == 0 else 3000),) + (1,) * tail, _groups(family)) == 0


@pytest.mark.parametrize("family", [0, 1, 2])
def test_requests_past_the_look(family):
    """More requests in the item than are looked at: from the queue."""
    assert _run(family, (1,) * 1025, _groups(family)) > 0
    assert _run(family, (1,) * 1024, _groups(family)) == 0
