"""The multi-kernel planner around the sizes at which its sorts take another
merge pass or width (blocks of 1024 keys, runs merged two to sixteen at a
time) and its sums another block: the served table, exactly, against the plan's
definition in numpy, with dropped requests, ties and tile slots."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd.batch import Batch  # noqa: E402
from paper_1108_0486_amd.streams import XorgensStreams  # noqa: E402

SEGMENT, LAST, MAX_TILES = 1, 2, 256


def _words(n, dtype):
    return n + (n & 1) if dtype == 2 else n


def _plan(reqs, num_streams, tile_words, slots):
    """(rows, group offsets): streams' requests grouped in stream order, a lone
    long request's tiles while they fit the slots, items by falling cost."""
    by = {}
    for r in reqs:
        if r[0] < num_streams and r[3] <= 2:
            by.setdefault(r[0], []).append(r)
    items, used = [], 0
    wants = []
    for s in sorted(by):
        g, want = by[s], 0
        if tile_words and len(g) == 1:
            want = -(-_words(g[0][1], g[0][3]) // tile_words)
            want = want if 1 < want <= MAX_TILES else 0
        wants.append(want)
    ends = np.cumsum(wants)
    for i, s in enumerate(sorted(by)):
        g, want, end = by[s], wants[i], int(ends[i])
        if want and end <= slots:
            st, n, off, dt = g[0]
            for k in range(want):
                nk = min(tile_words, n - k * tile_words)
                fl = SEGMENT | k << 8 | (end - want + k) << 16 | (LAST if k + 1 == want else 0)
                items.append((-_words(nk, dt) * (4 if dt == 2 else 1), i, k, [(st, nk, off + k * tile_words, dt, fl)]))
        else:
            cost = sum(_words(r[1], r[3]) * (4 if r[3] == 2 else 1) for r in g)
            items.append((-cost, i, 0, [tuple(r) + (0,) for r in g]))
    items.sort(key=lambda it: it[:3])
    rows = [r for it in items for r in it[3]]
    return rows, [0] + np.cumsum([len(it[3]) for it in items]).tolist()


@pytest.mark.parametrize("slots", [0, 900])
@pytest.mark.parametrize("num_reqs", [3300, 4097, 7000, 8192, 8193, 15000, 16384, 16385, 40000, 70000, 131073])
def test_large_plan_is_the_defined_one(num_reqs, slots):
    rng = np.random.default_rng(num_reqs + slots)
    if num_reqs + slots <= 4096:
        num_reqs += 4096
    S, L = num_reqs // 2 + 60, 4096
    stream = rng.integers(0, num_reqs // 2, num_reqs)
    n = rng.integers(0, 24, num_reqs)                     # many ties
    dtype = rng.integers(0, 3, num_reqs)
    dtype[rng.integers(0, num_reqs, 20)] = 3              # dropped
    stream[rng.integers(0, num_reqs, 20)] = S + 7         # dropped
    stream[: num_reqs // 50] = 11                         # one long group
    lone = rng.permutation(num_reqs)[:50]                 # lone long ones on streams of their own
    stream[lone], n[lone] = num_reqs // 2 + 1 + np.arange(50), rng.integers(5000, 150000, 50)
    off = np.concatenate([[0], np.cumsum(n)])
    reqs = [(int(stream[i]), int(n[i]), int(off[i]), int(dtype[i])) for i in range(num_reqs)]
    kw = {"tile_words": L, "max_tiles": slots} if slots else {}
    for order in (reqs, [r for r in reversed(reqs)]):
        gs = XorgensStreams(S, seed=5)
        b = Batch(gs, order, int(off[-1]), **kw)
        for _ in range(2):                                # the plan in scratch that a plan has used
            b.run()
            rows, groups = b.served_plan()
            want_rows, want_groups = _plan(order, S, L if slots else 0, slots)
            assert [int(g) for g in groups] == want_groups
            assert [tuple(int(v) for v in r) for r in rows] == want_rows
            assert b.error_flag() == 1


def test_all_dropped_and_none():
    gs = XorgensStreams(8, seed=5)
    b = Batch(gs, [(9, 4, 0, 0)] * 5000, 8)
    b.run()
    rows, groups = b.served_plan()
    assert len(rows) == 0 and [int(g) for g in groups] == [0] and b.error_flag() == 1
    good = Batch(gs, [(i % 8, 1, i, 0) for i in range(5000)], 5000)
    good.run()
    assert len(good.served_plan()[0]) == 5000 and good.error_flag() == 0


def test_large_plan_with_the_most_passes():
    """2^20 keys (ten doublings of runs of 1024): each stream's requests in
    table order, items by falling cost."""
    num_reqs, S = 600001, 300000
    rng = np.random.default_rng(9)
    stream, n = rng.integers(0, S, num_reqs), rng.integers(0, 5, num_reqs)
    off = np.concatenate([[0], np.cumsum(n)])
    gs = XorgensStreams(S, seed=5)
    b = Batch(gs, [(int(stream[i]), int(n[i]), int(off[i]), 0) for i in range(num_reqs)], int(off[-1]))
    b.run()
    rows, groups = b.served_plan()
    order = np.argsort(stream, kind="stable")
    first = np.flatnonzero(np.r_[True, np.diff(stream[order]) != 0])
    cost = np.add.reduceat(n[order], first)
    want = [order[a:z] for a, z in zip(first, np.r_[first[1:], num_reqs])]
    at = np.argsort(-cost, kind="stable")
    flat = np.concatenate([want[g] for g in at])
    got = np.array([[int(v) for v in r[:3]] for r in rows])
    assert (got == np.stack([stream[flat], n[flat], off[flat]], 1)).all()
    assert [int(g) for g in groups] == [0] + np.cumsum([len(want[g]) for g in at]).tolist()
