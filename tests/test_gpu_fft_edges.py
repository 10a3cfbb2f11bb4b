"""The latent at the edges of the FFT passes' ranges (the longest rows and
columns, odd and short grids, strips and rows that end inside a workgroup),
against a float64 division with the call's own kernels; frames with a pitch are
read up to their width and latents written up to theirs."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def smooth7(n):
    while True:
        r = n
        for p in (2, 3, 5, 7):
            while r % p == 0:
                r //= p
        if r == 1:
            return n
        n += 1


def blurred(m, n, k1, k2, seed):
    r = np.random.default_rng(seed)
    L = r.random((m, n))
    out = []
    for k in (k1, k2):
        K = r.random((k, k)) + 0.1
        K /= K.sum()
        s = (m + k - 1, n + k - 1)
        out.append(np.fft.irfft2(np.fft.rfft2(L, s) * np.fft.rfft2(K, s), s))
    return out


def division(b1, b2, K1, K2, m, n, lam):
    s = (smooth7(max(b1.shape[0], b2.shape[0])), smooth7(max(b1.shape[1], b2.shape[1])))
    B1, B2, F1, F2 = (np.fft.rfft2(np.asarray(x, float), s) for x in (b1, b2, K1, K2))
    q = (F1.conj() * B1 + F2.conj() * B2) / (abs(F1) ** 2 + abs(F2) ** 2 + lam)
    return np.fft.irfft2(q, s)[:m, :n]


@pytest.mark.parametrize("single", [True, False])
@pytest.mark.parametrize("m,n,k1,k2", [
    (11, 2040, 9, 4),     # rows of 2048: one half-spectrum entry beyond four a thread
    (2037, 9, 12, 5),     # columns of 2048
    (725, 30, 11, 3),     # an odd column length, 735
    (31, 723, 5, 7),      # an odd row length, 729
    (3, 300, 2, 3), (300, 3, 3, 2), (6, 6, 2, 2), (257, 513, 15, 13),
])
def test_latent_at_edges(single, m, n, k1, k2):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dtype = torch.float32 if single else torch.float64
    lam = 0.1
    frames = []
    for b in blurred(m, n, k1, k2, 3):
        big = torch.full((b.shape[0], b.shape[1] + 3), float("nan"), dtype=dtype, device="cuda")
        big[:, :-3] = torch.as_tensor(b, dtype=dtype)
        frames.append(big[:, :-3])
    L, K1, K2 = P.deblur(*frames, m, n, lam=lam)
    b1, b2 = (f.cpu().numpy() for f in frames)
    ref = division(b1, b2, K1.cpu().numpy(), K2.cpu().numpy(), m, n, lam)
    # a transform adds a few roundings a pass; the division amplifies those of
    # the kernels' spectra (k-term sums, k <= 15, of terms that add up to c) by
    # at most 1 / lam in the numerator and twice that in the denominator
    c = max(1.0, float(K1.abs().sum()), float(K2.abs().sum()))
    tol = (3 * 20 + 3 * 15 * c / lam) * 2.0 ** (-24 if single else -53)
    rms = lambda x: np.sqrt((np.asarray(x, float) ** 2).mean())
    assert rms(L.cpu().numpy() - ref) <= tol * rms(b1)


@pytest.mark.parametrize("single", [True, False])
def test_strip_width_of_a_mixed_batch(single):
    """Columns from 10 to 2048 entries and few to many strips in one launch: each
    frame gets the bits of its own call, whose strips have another width."""
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dtype = torch.float32 if single else torch.float64
    frames = []
    for s, (m, n) in enumerate([(2037, 20), (6, 700), (300, 301), (64, 64)] + 4 * [(257, 130)]):
        frames.append([torch.as_tensor(b, dtype=dtype, device="cuda") for b in blurred(m, n, 5, 4, s)] + [m, n])
    for part in (frames, frames[2:]):
        Ls, K1s, K2s, _ = P.deblur_batch(part, lam=1e-2)
        for f, L, K1, K2 in zip(part, Ls, K1s, K2s):
            assert all(torch.equal(x, y) for x, y in zip((L, K1, K2), P.deblur(*f, lam=1e-2)))


@pytest.mark.parametrize("rows", [1290, 1930])
def test_evaluation_of_long_items(rows):
    """Fused items of more than eight rows evaluate them in parts: the bits of
    the split pass, which takes one row at a time."""
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    r = np.random.default_rng(rows)
    frames = [[torch.as_tensor(r.random((3, rows + k - 1, 20 + k - 1)), dtype=torch.float32, device="cuda")
               for k in (5, 4)] + [rows, 20] for _ in range(4)]
    Ls, K1s, K2s, _ = P.deblur_batch(frames, lam=1e-2)
    for f, L, K1, K2 in zip(frames, Ls, K1s, K2s):
        assert all(torch.equal(x, y) for x, y in zip((L, K1, K2), P.deblur(*f, lam=1e-2)))


@pytest.mark.parametrize("single", [True, False])
@pytest.mark.parametrize("k1,k2", [(1, 2), (16, 15)])
def test_kernel_row_transforms_in_either_launch(single, k1, k2):
    """A call whose strips all run at once forms the kernels' row transforms in
    its column pass, one with more strips in a launch before it: the same bits."""
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dtype = torch.float32 if single else torch.float64
    frames = [[torch.as_tensor(b, dtype=dtype, device="cuda") for b in blurred(130, 390, k1, k2, s)] + [130, 390]
              for s in range(4)]
    Ls, K1s, K2s, _ = P.deblur_batch(12 * frames, lam=1e-2)
    for f in (0, 1, 2, 3, 45):
        assert all(torch.equal(x, y) for x, y in zip((Ls[f], K1s[f], K2s[f]), P.deblur(*frames[f % 4], lam=1e-2)))
