"""The one-workgroup planner around the sizes at which its workgroup, and the
elements per thread, change (256, 512, 1024, 2048 and 4096), with and without
tile slots: the plan against its rules and the multi-kernel planner's."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from test_gpu_batch import _check_plan, _plan_pair  # noqa: E402


@pytest.mark.parametrize("slots", [0, 55])
@pytest.mark.parametrize("elems", [56, 64, 65, 255, 256, 257, 511, 512, 513, 1023, 1025, 2047, 2048, 2049, 4095])
def test_plan_at_size_edges(elems, slots):
    rng = np.random.default_rng(elems)
    num_reqs, S, L = elems - slots, 400, 4096
    reqs, off = [], 0
    for i in range(num_reqs):
        long = slots and i % 37 == 5
        n = int(rng.integers(2 * L, 5 * L)) if long else int(rng.integers(0, 90))
        stream = 399 - i // 37 if long else int(rng.integers(0, 250))   # long ones alone on their streams
        reqs.append((max(250, stream) if long else stream, n, off, int(rng.integers(0, 3)) if i % 11 else i % 4))
        off += n
    small = {"tile_words": L, "max_tiles": slots} if slots else {}
    (plan_a, err_a, out_a, st_a), (plan_b, err_b, out_b, st_b) = _plan_pair(
        reqs, off, S, 13, small, {"tile_words": L if slots else 1 << 30, "max_tiles": slots if slots else 4096})
    assert plan_a == plan_b and err_a == err_b == int(any(r[3] > 2 for r in reqs))
    assert (out_a == out_b).all() and all((x == y).all() for x, y in zip(st_a, st_b))
    rows, groups = plan_a
    _check_plan([r for r in reqs if r[3] <= 2], rows, groups, S, **({"tile_words": L} if slots else {}))
