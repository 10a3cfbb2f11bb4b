"""The double-double forms' workgroup eigen-solver at the edges of its
instances (solve orders 16, 24, 32, 40 and 64 and one past each), against the
FP64 oracle."""

import numpy as np
import pytest

import synth
from oracle import cbp as orc

pytestmark = pytest.mark.gpu

rel = lambda a, b: float(np.linalg.norm(a - b) / np.linalg.norm(b))   # noqa: E731


def frame(torch, k1, k2, m=96, n=88):
    r = synth.rng_for(77, k1, k2)
    L = synth.uniform_scene(r, m, n)
    K1, K2 = synth.draw_coprime_pair(r, k1, k2, "uniform")
    B1, B2 = synth.blur_pair(r, L, K1, K2, 0.0)
    return B1, B2, torch.as_tensor(B1, device="cuda"), torch.as_tensor(B2, device="cuda"), m, n


# (k1, k2): sample order k1 + k2, scale order 2 max(k1, k2)
@pytest.mark.parametrize("k1,k2", [(1, 1), (1, 2), (8, 8), (8, 9), (12, 12), (13, 12), (16, 16), (17, 16), (20, 20),
                                   (21, 20)])
def test_orders(k1, k2):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    B1, B2, b1, b2, m, n = frame(torch, k1, k2)
    K1, K2, diag = P.recover_kernels(b1, b2, m, n, diag=True)
    G1, G2 = P.recover_kernels(b1, b2, m, n)
    R1, R2 = orc.recover_kernels(B1, B2, m, n)
    assert diag["flags"] == 0
    assert max(rel(K1.cpu().numpy(), R1), rel(K2.cpu().numpy(), R2)) <= 1e-6     # the FP64 form's bound
    # the diagnostics (second eigenvalue, Rayleigh quotient) change no result
    assert rel(G1.cpu().numpy(), K1.cpu().numpy()) <= 1e-12


def test_orders_share_a_launch():
    """A frame's kernels do not depend on the instance that a larger frame of its batch asks for."""
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    frames = [frame(torch, *k)[2:] for k in ((3, 4), (9, 11), (15, 17), (21, 20))]
    _, K1s, K2s, _ = P.deblur_batch(frames, lam=1e-6)
    for f, A, B in zip(frames, K1s, K2s):
        _, K1, K2 = P.deblur(*f, lam=1e-6)
        assert torch.equal(A, K1) and torch.equal(B, K2)


# smallest eigenvalues from rounding level (no noise) to a good part of the largest (noise alone)
@pytest.mark.parametrize("noise", [0.0, 1e-6, 1e-3, 1e-1, None])
def test_size_of_smallest_eigenvalue(noise):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    B1, B2, _, _, m, n = frame(torch, 7, 5)
    r = np.random.default_rng(5)
    B1, B2 = (r.standard_normal(B.shape) if noise is None else B + noise * r.standard_normal(B.shape) for B in (B1, B2))
    K1, K2 = P.recover_kernels(torch.as_tensor(B1, device="cuda"), torch.as_tensor(B2, device="cuda"), m, n)
    R1, R2 = orc.recover_kernels(B1, B2, m, n)
    assert max(rel(K1.cpu().numpy(), R1), rel(K2.cpu().numpy(), R2)) <= 1e-6     # the FP64 form's bound
