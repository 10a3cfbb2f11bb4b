"""The two forms of the forward row pass (single rows with a separate column
fold in small calls, residue items that fold as they go in large ones) and the
column fold's four-column groups give the same bits, whatever the frames'
alignment."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def pair(torch, seed, m, n, k1, k2, ch, dtype):
    r = np.random.default_rng(seed)
    shape = () if ch == 1 else (ch,)
    return [torch.as_tensor(r.random(shape + (m + k - 1, n + k - 1)), dtype=dtype, device="cuda") for k in (k1, k2)] + [m, n]


@pytest.mark.parametrize("single", [True, False])
@pytest.mark.parametrize("m,n,k1,k2,ch,count", [(150, 131, 5, 7, 1, 24), (97, 300, 9, 9, 3, 12), (33, 255, 1, 2, 1, 30)])
def test_large_batch_equals_single_calls(single, m, n, k1, k2, ch, count):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dtype = torch.float32 if single else torch.float64
    frames = [pair(torch, s, m, n, k1, k2, ch, dtype) for s in range(count)]
    Ls, K1s, K2s, _ = P.deblur_batch(frames, lam=1e-3)
    for f in (0, count // 2, count - 1):
        L, K1, K2 = P.deblur(*frames[f], lam=1e-3)
        assert torch.equal(K1s[f], K1) and torch.equal(K2s[f], K2) and torch.equal(Ls[f], L)


@pytest.mark.parametrize("single", [True, False])
@pytest.mark.parametrize("shift", [1, 2, 3])
def test_misaligned_frames(single, shift):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dtype = torch.float32 if single else torch.float64
    b1, b2, m, n = pair(torch, 7, 60, 259, 5, 4, 1, dtype)

    def moved(b):
        big = torch.full((b.shape[0], b.shape[1] + 5), 3.0, dtype=dtype, device="cuda")
        big[:, shift:shift + b.shape[1]] = b
        return big[:, shift:shift + b.shape[1]]

    a = P.deblur(b1, b2, m, n, lam=1e-3)
    c = P.deblur(moved(b1), moved(b2), m, n, lam=1e-3)
    assert all(torch.equal(x, y) for x, y in zip(a, c))
    assert all(torch.equal(x, y) for x, y in zip(a[1:], P.recover_kernels(moved(b1), moved(b2), m, n)))
    for x, y in zip(P.eval_unit_circle(b1, 7), P.eval_unit_circle(moved(b1), 7)):
        assert torch.equal(x, y)
