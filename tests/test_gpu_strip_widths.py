"""The column pass with strips of 8, 4 and 2 columns shared by frames of every
filter group and of short and long columns in one launch: each frame gets the
bits of its own call, whose strips are one column wide.  And the fused row pass
at the smallest sample count, which a batch must be large to reach.

The widths are those of the host's rule: the widest that every frame's strip
fits in registers and LDS, halved until the call has 512 strips."""

import numpy as np
import pytest

torch = pytest.importorskip("torch")
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


def group(N):
    return next((g for g in (4, 5, 7, 3) if N % g == 0), 1)


def width(shapes, esize):
    """Strip width of a call; shapes: (rows, columns, channels) of the larger frame of each pair."""
    hx = [smooth7(w) // 2 + 1 for _, w, _ in shapes]
    cw = 8
    while cw > 1 and (any(cw * smooth7(h) > 512 * 72 // (2 * esize) for h, _, _ in shapes) or
                      sum(-(-x // cw) * c for x, (_, _, c) in zip(hx, shapes)) < 512):
        cw //= 2
    return cw


# rows of the larger frame: 7, 9, 10, 12, 14 (filter groups 7, 3, 5, 4, 7), then longer ones up to the width's longest
@pytest.mark.parametrize("single,rows,want", [
    (True, [7, 9, 10, 12, 14, 45, 63, 288, 441, 576], 8), (False, [7, 9, 10, 12, 14, 45, 63, 105, 243, 288], 8),
    (True, [7, 9, 10, 12, 245, 875, 1152], 4), (False, [7, 9, 10, 12, 245, 441, 576], 4),
    (True, [7, 9, 12, 1715, 2025, 2048], 2), (False, [7, 9, 12, 735, 875, 1152], 2)])
def test_wide_strips_of_a_mixed_batch(single, rows, want):
    import paper_1203_4874_amd as P
    dtype, esize = (torch.float32, 4) if single else (torch.float64, 8)
    r = np.random.default_rng(want)
    k1, k2 = 5, 4
    frames, shapes = [], []
    for i, H in enumerate(rows):
        m, n, ch = H - k1 + 1, (700, 333, 810, 96)[i % 4] + i, 1 + i % 2
        shapes.append((H, n + k1 - 1, ch))
        shape = () if ch == 1 else (ch,)
        frames.append([torch.as_tensor(r.random(shape + (m + k - 1, n + k - 1)), dtype=dtype, device="cuda")
                       for k in (k1, k2)] + [m, n])
    count = 1
    while sum(-(-(smooth7(w) // 2 + 1) // want) * c for _, w, c in shapes) * count < 512:
        count += 1
    assert width(count * shapes, esize) == want and all(width([s], esize) == 1 for s in shapes)
    assert {group(smooth7(H)) for H in rows} >= {3, 4, 7}
    d = P.Deblurrer(2060, 840, 5, 2, count * len(rows), P.Precision.MIXED if single else P.Precision.FP64)
    Ls, K1s, K2s, _ = d.deblur_batch(count * frames, lam=1e-2)
    for f, frame in enumerate(frames):
        own = P.deblur(*frame, lam=1e-2)
        for at in (f, f + (count - 1) * len(rows)):
            assert all(torch.equal(x, y) for x, y in zip((Ls[at], K1s[at], K2s[at]), own))


@pytest.mark.parametrize("single,m,n,k1,k2,count", [(True, 33, 255, 1, 2, 210), (False, 130, 255, 1, 2, 128),
                                                     (True, 120, 40, 1, 1, 210)])
def test_fused_rows_of_few_samples(single, m, n, k1, k2, count):
    """Sample counts 1 and 2: 32 and 16 rows a residue and fold group."""
    import paper_1203_4874_amd as P
    dtype = torch.float32 if single else torch.float64
    r = np.random.default_rng(7)
    frames = [[torch.as_tensor(r.random((m + k - 1, n + k - 1)), dtype=dtype, device="cuda") for k in (k1, k2)] + [m, n]
              for _ in range(4)]
    with P.profile() as p:
        Ls, K1s, K2s, _ = P.deblur_batch([frames[f % 4] for f in range(count)], lam=1e-3)
        torch.cuda.synchronize()
    assert p.result["fold_cols"][1] == 1                       # the fused form
    for f in (0, 1, count // 2, count - 1):
        with P.profile() as p:
            own = P.deblur(*frames[f % 4], lam=1e-3)
            torch.cuda.synchronize()
        assert p.result["fold_cols"][1] == 0                   # the split form
        assert all(torch.equal(x, y) for x, y in zip((Ls[f], K1s[f], K2s[f]), own))
