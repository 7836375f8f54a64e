"""Batches whose groups hold several requests, at the lengths where a request
ends inside, at or past a chunk of its stream, in tables that few and that many
wavefronts serve: every request's values are those the same stream gives when
it is asked for them one after another, and the end states agree."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from oracle import oracle as O  # noqa: E402
from paper_1108_0486_amd.batch import Batch  # noqa: E402
from paper_1108_0486_amd.streams import XorgensStreams  # noqa: E402

EDGES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 513, 1025]


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("lone", [False, True])     # one request to a stream
@pytest.mark.parametrize("streams", [1, 2, 7, 64, 1501, 3001, 13001])
@pytest.mark.parametrize("family", [0, 1, 2])
def test_groups_continue_their_stream(streams, family, lone, mixed):
    rng = np.random.default_rng(streams + family)
    k = streams if lone else max(60, 3 * streams)
    stream = rng.permutation(streams) if lone else rng.integers(0, streams, k)
    n = rng.choice(EDGES, k)
    dtype = rng.integers(0, 3, k) if mixed else np.full(k, streams % 3)
    off = np.concatenate([[0], np.cumsum(n)])
    gs = XorgensStreams(streams, seed=21, family=family)
    b = Batch(gs, [(int(stream[i]), int(n[i]), int(off[i]), int(dtype[i])) for i in range(k)], int(off[-1]))
    ref = XorgensStreams(streams, seed=21, family=family)
    wide = family == 2
    real = torch.float64 if wide else torch.float32
    names = ("u64", "f64", "normal_f64") if wide else ("u32", "f32", "normal")
    check = range(k) if streams < 100 else [i for i in range(k) if stream[i] in (0, 5, streams - 1)]
    for _ in range(2):
        b.run()
        assert b.error_flag() == 0
        for i in check:
            if n[i]:
                got = b.out[int(off[i]):int(off[i + 1])]
                want = getattr(ref, names[dtype[i]])(int(n[i]), first=int(stream[i]), count=1).view(-1)
                got = got if dtype[i] == 0 else got.view(real)
                assert torch.equal(got, want.view(got.dtype) if dtype[i] == 0 else want), i
    per = gs.state.numel() // streams
    for s in sorted({int(stream[i]) for i in check}):
        assert torch.equal(gs.state[s * per:(s + 1) * per], ref.state[s * per:(s + 1) * per]), s


def test_words_of_a_group_are_the_oracles():
    lengths = EDGES * 2
    off = np.concatenate([[0], np.cumsum(lengths)])
    gs = XorgensStreams(3, seed=8)
    b = Batch(gs, [(1, int(m), int(off[i]), 0) for i, m in enumerate(lengths)], int(off[-1]))
    b.run()
    want = O.OracleStreams(8, 3, params=O.PAPER).u32(int(off[-1]))[1]
    assert (b.out.cpu().numpy().view(np.uint32) == want).all()
