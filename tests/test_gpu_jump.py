"""The two forms of the matrix-core jump: a workgroup per stream (up to four
streams per compute unit) and a wavefront per stream (beyond), with more
streams than wavefronts in the grid, against each other and the oracle."""
import numpy as np
import pytest

from gpu_helpers import needs_gpu
from oracle import oracle as O

pytestmark = [pytest.mark.gpu, needs_gpu]

torch = pytest.importorskip("torch")

from paper_1108_0486_amd.streams import XorgensStreams  # noqa: E402


@pytest.mark.parametrize("per_cu,more", [(4, 1), (8, 3), (16, 5), (33, 0)])
@pytest.mark.parametrize("J", [1 << 15, (1 << 40) + 777, 2**64 - 1])
def test_jump_forms_agree(per_cu, more, J):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    S = per_cu * cus + more
    a, b = XorgensStreams(S, seed=21), XorgensStreams(S, seed=21)
    a.skip(J)                                        # a wavefront per stream
    for first in range(0, S, 4 * cus):               # a workgroup per stream
        b.skip(J, first=first, count=min(4 * cus, S - first))
    assert torch.equal(a.state, b.state)
    rows = [0, 7, 8, S // 2, S - 1]
    ref = O.OracleStreams(21, S).subset(rows)
    g = O.poly_to_words(O.z_pow_mod(J, O.charpoly(O.PAPER)), 64)
    ring, weyl, pos = a.host_state(rows)
    for j in range(len(rows)):
        assert (ring[j] == O.xpart_jump_poly(O.PAPER, ref.ring[j], g)).all(), rows[j]
    step = np.uint64(J % 2**32) * np.uint64(O.PAPER.omega)
    assert (weyl == ((ref.weyl.astype(np.uint64) + step) % np.uint64(2**32)).astype(np.uint32)).all()
    assert (pos == np.uint64(J)).all()


def test_jump_of_one_bit_states():
    """States with a single bit set, and all bits set: every column of the
    jump's matrix counts, and no sum over them is lost to rounding."""
    J = (1 << 30) + 12345
    S = 130
    gs = XorgensStreams(S, seed=1)
    words = torch.zeros(S, 132, dtype=torch.int32)
    rng = np.random.default_rng(5)
    bits = rng.choice(4096, size=S - 1, replace=False)
    for i, bit in enumerate(bits):
        words[i, bit // 32] = int(np.uint32(1 << (int(bit) % 32)).view(np.int32))
    words[S - 1, :128] = -1
    gs.state.copy_(words.reshape(-1))
    ring0, _, _ = gs.host_state()
    gs.skip(J)
    ring, _, _ = gs.host_state()
    g = O.poly_to_words(O.z_pow_mod(J, O.charpoly(O.PAPER)), 64)
    for i in range(S):
        assert (ring[i] == O.xpart_jump_poly(O.PAPER, ring0[i], g)).all(), i


@pytest.mark.parametrize("family,params", [(1, O.R64), (2, O.W64)])
@pytest.mark.parametrize("per_cu,more", [(1, 1), (6, 5), (20, 3)])
def test_member_jump_forms_agree(family, params, per_cu, more):
    """The further members: a few pairs of streams per workgroup, and beyond
    that a wavefront per pair, with one stream alone in the last pair."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    S, J = per_cu * cus + more, (1 << 40) + 777
    a, b = XorgensStreams(S, seed=21, family=family), XorgensStreams(S, seed=21, family=family)
    a.skip(J)
    for first in range(0, S, cus + 1):
        b.skip(J, first=first, count=min(cus + 1, S - first))
    assert torch.equal(a.state, b.state)
    rows = [0, 1, S // 2, S - 1]
    one = (lambda i: O.OracleStreams64(21 + i, 1, O.W64)) if family == 2 else (
        lambda i: O.OracleStreams(21 + i, 1, params=O.R64))
    g = O.poly_to_words(O.z_pow_mod(J, O.charpoly(params)), params.n // 64)
    ring, weyl, pos = a.host_state(rows)
    for j in range(len(rows)):
        want = np.asarray(O.xpart_jump_poly(params, one(rows[j]).ring[0], g)).astype(ring.dtype)
        assert (ring[j] == want).all(), rows[j]
    assert (pos == np.uint64(J)).all()
