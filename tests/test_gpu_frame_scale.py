"""Frames scaled by a power of two, which scales every sum up to the Gram
exactly: the kernels and the size search are those of the frames themselves,
also where the squares of the Gram's entries, or of the roundings that a
singular Gram leaves, fall out of double's range; a Gram beyond the solver's
own range (norms from 2^-464 to 2^511) gives zero kernels, a zero latent and
the flags of a solve that failed."""

import numpy as np
import pytest

import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def frames(e, seed=11, m=60, n=52, k1=6, k2=5):
    r = synth.rng_for(seed, k1, k2)
    L = synth.uniform_scene(r, m, n)
    K1, K2 = synth.draw_coprime_pair(r, k1, k2, "uniform")
    B1, B2 = synth.blur_pair(r, L, K1, K2, 0.0)
    return [torch.as_tensor(np.ldexp(B, e), device="cuda") for B in (B1, B2)] + [m, n]


def deblurred(P, e):
    b1, b2, m, n = frames(e)
    d = P.Deblurrer(max(b1.shape[0], b2.shape[0]), max(b1.shape[1], b2.shape[1]), 6, diag=True)
    L, K1, K2 = d.deblur(b1, b2, m, n, lam=1e-6)
    return L, K1, K2, d.read_diag()["flags"]


# the Gram's norm is about 2^(2 e + 17)
@pytest.mark.parametrize("e", [-233, -200, 230])
def test_kernels_of_scaled_frames(e):
    import paper_1203_4874_amd as P
    L0, A0, B0, f0 = deblurred(P, 0)
    L, A, B, f = deblurred(P, e)
    assert f == f0 == 0
    for x, y in ((A, A0), (B, B0), (L * 2.0 ** -e, L0)):
        assert float((x - y).norm()) <= 1e-12 * float(y.norm())


@pytest.mark.parametrize("e", [-256, -299, -332, -465, 256, 300])
def test_grams_out_of_range(e):
    import paper_1203_4874_amd as P
    L, A, B, flags = deblurred(P, e)
    assert flags == 15
    assert not A.any() and not B.any() and not L.any()


@pytest.mark.parametrize("e", [-255, -233, 0, 230])
def test_size_search_of_scaled_frames(e):
    import paper_1203_4874_amd as P
    r, r0 = (P.estimate_kernel_sizes(*frames(x)[:2], 3, 10, 1) for x in (e, 0))
    assert (r["k1"], r["k2"], r["flags"]) == (6, 5, 0)
    assert np.abs(r["scores"] - r0["scores"]).max() <= 1e-9
