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


def _table(family, reqs, streams):
    """The queue counter a batch of (stream, n, dtype) leaves, its values checked stream by stream."""
    off = np.concatenate([[0], np.cumsum([n for _, n, _ in reqs])])
    a, b = XorgensStreams(streams, seed=5, family=family), XorgensStreams(streams, seed=5, family=family)
    batch = Batch(a, [(s, n, int(o), d) for (s, n, d), o in zip(reqs, off)], int(off[-1]))
    batch.out.zero_()
    batch.run(tune=SHAPE)
    words = (b.u64 if family == 2 else b.u32)(int(off[-1]) // streams * 2)
    at = [0] * streams
    rows = [i for i, (_, _, d) in enumerate(reqs) if d == 0]
    for i, (s, n, d) in enumerate(reqs):
        if i in rows[:40] or i in rows[-40:]:
            assert torch.equal(batch.out[off[i]:off[i + 1]], words[s, at[s]:at[s] + n]), i
        at[s] += n + (n & 1 if d == 2 else 0)
    assert a.host_state()[2].tolist() == at and batch.error_flag() == 0
    return int(batch.scratch[0].item())


@pytest.mark.parametrize("family", [1, 2])
def test_one_uneven_pair_does_not_turn_the_table(family):
    """Requests of 6000 words, dealt where pairs run evenly and taken from the
    queue where they do not."""
    G = _groups(family)
    single = [(s, 6000, 0) for s in range(G)]
    assert _table(family, single, G) == 0
    assert _table(family, [(0, 3100, 0), (0, 3000, 0)] + single[1:], G) == 0
    # A small pair of two types ends before the others; the largest of two types ends last.
    assert _table(family, single[:-2] + [(G - 2, 800, 0), (G - 1, 200, 2)], G) == 0
    assert _table(family, [(0, 6000, 0), (1, 1500, 2)] + single[2:], G) > 0
    # Half of the pairs of two types.
    assert _table(family, [(s, 6000, 0) if s % 4 else (s, 1500, 2) for s in range(G)], G) > 0
