"""The encoder's draws of more frames than one launch of probes can hold (fewer
than 2^32 threads): the frames on both sides of every turn's end are those of a
call of their own."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_more_frames_than_a_launch_holds():
    import paper_1203_4874_amd as P
    k1, k2, S, seed, first = 2, 3, 3, 77, 5
    per = 2 * S * 128                                  # probe threads a frame
    count = 2 ** 32 // per + 1
    K1s, K2s, att, mr = P.draw_kernel_pairs(seed, first, count, k1, k2)
    turn = 2 ** 23 // S                                # frames of a turn
    for at in (0, turn - 3, 2 * turn - 3, 2 ** 22 - 3, count - 6):
        n = min(6, count - at)
        A, B, a, r = P.draw_kernel_pairs(seed, first + at, n, k1, k2)
        assert torch.equal(K1s[at:at + n], A) and torch.equal(K2s[at:at + n], B)
        assert np.array_equal(att[at:at + n], a) and np.array_equal(mr[at:at + n], r)
    assert att.min() >= 0 and mr.min() > 1e-12 and mr.max() < 1.0
