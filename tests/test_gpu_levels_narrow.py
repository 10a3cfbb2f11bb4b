"""The 8-bit conversions of pitched and misaligned images of few columns, whose
rows share workgroups: byte for byte against the oracle at the widths where the
lanes a row change, on heights that end inside a workgroup and one that takes
the grid round twice; and such an image costs about what its bytes do."""

import numpy as np
import pytest

from oracle import encoder as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(3, 1025, 1), (2, 513, 2), (1, 1000, 3), (70, 5), (3, 129, 8), (257, 9), (2, 67, 63), (2, 33, 64),
                                   (40, 65), (9, 255), (2, 9, 256), (4, 257), (2, 5, 511), (3, 512), (3, 513),
                                   (2, 1025), (262145, 129)])
@pytest.mark.parametrize("single", [True, False])
def test_narrow_layouts(shape, single):
    import paper_1203_4874_amd as P
    if shape[0] > 100000 and not single:
        pytest.skip("one type is enough for the grid's second round")
    dt, npd = (torch.float32, np.float32) if single else (torch.float64, np.float64)
    B = (1.2 * np.random.default_rng(len(shape)).random(shape) - 0.1).astype(npd)

    def image(dtype, fill):   # a gap of two elements between rows
        full = torch.full(shape[:-1] + (shape[-1] + 2,), fill, dtype=dtype, device="cuda")
        return full, full[..., :shape[-1]]

    _, src = image(dt, 9.0)
    src.copy_(torch.as_tensor(B))
    qall, q = image(torch.uint8, 77)
    P.quantize(src, 1, out=q)
    want = orc.quantize(B, 1)
    assert np.array_equal(q.cpu().numpy(), want)
    assert bool((qall[..., shape[-1]:] == 77).all())
    oall, out = image(dt, 9.0)
    P.dequantize(q, out=out)
    assert np.array_equal(out.cpu().numpy(), orc.dequantize(want, npd))
    assert bool((oall[..., shape[-1]:] == 9.0).all())


@pytest.mark.parametrize("rows,cols", [(1000000, 8), (1000000, 1), (60000, 200)])
def test_narrow_rows_cost_their_bytes(rows, cols):
    """Against the same number of elements as one run.  A row of c FP32 and c bytes at a pitch of c + 1 is
    at most the next whole 32-byte sectors, under twice the bytes from c = 1 on; a workgroup a row costs ten
    times and more."""
    import paper_1203_4874_amd as P

    def best(src, q):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ts = []
        for _ in range(12):
            ev[0].record()
            for _ in range(4):
                P.quantize(src, 0, out=q)
            ev[1].record()
            torch.cuda.synchronize()
            ts.append(ev[0].elapsed_time(ev[1]))
        return min(ts)

    n = max(rows * cols, 8000000)   # (a run short enough to be all launch would hide the difference)
    run = best(torch.zeros((1, n), device="cuda"), torch.zeros((1, n), dtype=torch.uint8, device="cuda"))
    narrow = best(torch.zeros((rows, cols + 1), device="cuda")[:, :cols],
                  torch.zeros((rows, cols + 1), dtype=torch.uint8, device="cuda")[:, :cols])
    assert narrow <= 4.0 * run
