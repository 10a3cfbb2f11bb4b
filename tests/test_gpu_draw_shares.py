"""The encoder's draws where several kernels, or several frames' checks, share a
workgroup (kernels up to 8x8, an odd number of frames; 65536 frames and more):
every frame as the oracle draws it, and redraws among many frames."""

import numpy as np
import pytest

from oracle import encoder as enc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k1,k2,frames", [(8, 8, 1), (8, 8, 3), (1, 8, 5), (8, 9, 3), (2, 1, 7), (1, 1, 3)])
def test_small_kernels_bitwise(k1, k2, frames):
    import paper_1203_4874_amd as P
    K1s, K2s, att, _ = P.draw_kernel_pairs(9, 3, frames, k1, k2)
    for f in range(frames):
        R1, R2, a = enc.draw_pair(9, 3 + f, k1, k2)
        assert att[f] == a
        assert np.array_equal(K1s[f].cpu().numpy(), R1) and np.array_equal(K2s[f].cpu().numpy(), R2)


@pytest.mark.parametrize("count", [65537, 200001])
def test_many_frames(count):
    import paper_1203_4874_amd as P
    K1s, K2s, att, mr = P.draw_kernel_pairs(9, 0, count, 2, 2)
    assert np.count_nonzero(att) > 0     # three of these pairs are redrawn
    pick = np.unique(np.concatenate([np.argsort(mr)[:4], np.nonzero(att)[0][:4], [0, 63, 64, 65535, 65536, count - 1]]))
    for f in pick:
        A, B, a, r = P.draw_kernel_pairs(9, int(f), 1, 2, 2)
        assert torch.equal(K1s[f], A[0]) and torch.equal(K2s[f], B[0]) and att[f] == a[0] and mr[f] == r[0]
    assert att.min() >= 0 and mr.min() > 1e-12
