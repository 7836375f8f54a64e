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
