"""The 8-bit conversions on dense images (16 elements per thread: totals around
multiples of 16 and of a workgroup's 4096) and on pitched or misaligned ones,
byte for byte against the oracle."""

import numpy as np
import pytest

from oracle import encoder as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1), (3, 5), (4, 4), (1, 17), (64, 64), (63, 65), (2, 45, 91), (3, 32, 128)])
@pytest.mark.parametrize("single", [True, False])
@pytest.mark.parametrize("pad,shift", [(0, 0), (0, 1), (5, 0)])
def test_layouts(shape, single, pad, shift):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dt, npd = (torch.float32, np.float32) if single else (torch.float64, np.float64)
    B = (1.2 * np.random.default_rng(len(shape)).random(shape) - 0.1).astype(npd)

    def image(dtype, fill):
        # rows of shape[-1] + pad elements, starting `shift` elements into the buffer
        full = shape[:-1] + (shape[-1] + pad,)
        flat = torch.full((int(np.prod(full)) + shift,), fill, dtype=dtype, device="cuda")
        return flat, flat[shift:].view(full)[..., :shape[-1]]

    _, src = image(dt, 9.0)
    src.copy_(torch.as_tensor(B))
    qflat, q = image(torch.uint8, 77)
    P.quantize(src, 2, out=q)
    want = orc.quantize(B, 2)
    assert np.array_equal(q.cpu().numpy(), want)
    assert int((qflat == 77).sum()) == qflat.numel() - q.numel() + int((want == 77).sum())
    oflat, out = image(dt, 9.0)
    P.dequantize(q, out=out)
    assert np.array_equal(out.cpu().numpy(), orc.dequantize(want, npd))
    assert int((oflat == 9.0).sum()) == oflat.numel() - out.numel()
