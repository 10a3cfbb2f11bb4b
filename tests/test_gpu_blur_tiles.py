"""The encoder's blur at the edges of its 64 x 64 tiles and of its two launch
forms (both streams in one launch up to 8 x 8 kernels, one launch each above),
against the exact-order oracle within the rounding bound of the direct sum."""

import numpy as np
import pytest

from oracle import encoder as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k1,k2", [(1, 1, 1, 1), (64, 64, 1, 8), (57, 65, 8, 7), (56, 56, 9, 9), (63, 128, 2, 32),
                                       (65, 33, 32, 31), (130, 61, 16, 17)])
@pytest.mark.parametrize("ch,single", [(1, False), (2, True)])
def test_tiles(m, n, k1, k2, ch, single):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    dtype, u = (torch.float32, 2.0 ** -24) if single else (torch.float64, 2.0 ** -53)
    r = np.random.default_rng([m, n, k1, k2])
    L = torch.as_tensor(r.random((ch, m, n)), dtype=dtype, device="cuda")
    Ks = [r.random((k, k)) for k in (k1, k2)]
    Ks = [K / K.sum() for K in Ks]
    out = P.encode(L, *[torch.as_tensor(K, device="cuda") for K in Ks])
    for K, B in zip(Ks, out):
        k = K.shape[0]
        for c in range(ch):
            ref = orc.blur(L[c].double().cpu().numpy(), K)
            assert np.all(np.abs(B[c].double().cpu().numpy() - ref) <= (k * k + 2) * u * np.abs(ref) + 1e-300)
