"""The fused training step at the edges of its 64-row blocks and past its 256
workgroups (more rows than 256 blocks: a workgroup takes several), against the
oracle with the same bfloat16 rounding points."""

import numpy as np
import pytest

from oracle import learned as orl

pytestmark = pytest.mark.gpu

# Both sides round the same seven operands to bfloat16; they differ where an
# FP32 sum taken in another order falls on the other side of a rounding
# boundary (about 2^-15 of the entries, by u = 2^-8 each) and by the FP32
# sums themselves, far below the per-block bound 1e-2 used for 700 rows.
BOUND = 1e-2


@pytest.mark.parametrize("n", [1, 63, 64, 65, 128, 16384, 16385, 33000])
def test_gradients(n):
    torch = pytest.importorskip("torch")
    import paper_1203_4874_amd as P
    r = np.random.default_rng(n)
    q = {"W1": r.standard_normal((128, 32)) * 0.25, "b1": 0.1 * r.standard_normal(128),
         "W2": r.standard_normal((128, 128)) * 0.12, "b2": 0.1 * r.standard_normal(128),
         "W3": r.standard_normal((2, 128)) * 0.1, "b3": 0.1 * r.standard_normal(2)}
    q = {k: v.astype(np.float32).astype(np.float64) for k, v in q.items()}
    X = (-1.4 * r.random((n, 32))).astype(np.float32).astype(np.float64)
    T = np.stack([r.standard_normal(n), r.standard_normal(n) - 3.0], 1).astype(np.float32).astype(np.float64)
    st = P.MlpState(n)
    st.set_params(orl.pack(q).astype(np.float32))
    dev = [torch.as_tensor(v, dtype=torch.float32, device="cuda") for v in (X, T)]
    loss, g = st.gradients(*dev)
    lo, go = orl.loss_and_grad_bf16(q, X, T[:, 0], T[:, 1])
    assert abs(float(loss.item()) - lo) <= 1e-3 * abs(lo)
    gg = orl.unpack(g.cpu().numpy())
    for k in gg:
        assert np.linalg.norm(gg[k] - go[k]) <= BOUND * np.linalg.norm(go[k]), k
    # a training step sees the same gradient: its first Adam step is lr g / (|g| + eps)
    p0 = st.get_params().double()
    st.train_step(*dev, 1e-3, 1)
    gd = g.double()
    want = p0 - 1e-3 * gd / (gd.abs() + 1e-8)
    assert float((st.get_params().double() - want).abs().max()) <= 1e-3 * 2e-5 + 2.0 ** -23 * float(p0.abs().max())
