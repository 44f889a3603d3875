"""The fused training step against the NumPy reference at the batch sizes where it can go wrong: one row,
a workgroup's 64 rows and their neighbours, the most workgroups and several blocks of rows for each.  The
tolerance is the one that the router's own gradient test holds this comparison to."""
import numpy as np
import pytest

from oracle import router as ref
import paper_1711_00975_amd as csk

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("n", [1, 15, 63, 64, 65, 1000, 8192, 8193, 20_001])
def test_train_step_matches_the_reference(n):
    import torch
    print("train", n, flush=True)
    rng = np.random.default_rng(n)
    w = ref.unpack(rng.normal(0, 0.25, ref.N_PARAMS).astype(np.float32))
    w["W1"][:, 27:] = 0
    p = ref.pack(w)
    x = np.zeros((n, 32), np.float32)
    x[:, :27] = np.log1p(rng.poisson(3.0, (n, 27))).astype(np.float32)
    y = (rng.random(n) < 0.3).astype(np.float32)
    m = csk.MLP(seed=5, max_batch=n)
    try:
        m.set_params(p)
        loss = torch.zeros(1, dtype=torch.float32, device="cuda")
        lr = 1e-3
        m.train_step(_dev(x), _dev(y), lr, loss)
        g, want = m.grads(), ref.gradients(p, x, y)
        assert np.allclose(g, want, rtol=2e-3, atol=1e-6), np.max(np.abs(g - want))
        z = ref.forward(p, x)[0].astype(np.float64)
        ce = np.maximum(z, 0) - z * y + np.log1p(np.exp(-np.abs(z)))
        assert abs(loss.item() - ce.mean()) <= 1e-4 * max(1.0, ce.mean())
        # Adam's first step from these gradients
        lr_t = lr * np.sqrt(1 - 0.999) / (1 - 0.9)
        g64 = g.astype(np.float64)
        step = lr_t * 0.1 * g64 / (np.sqrt(0.001 * g64 * g64) + 1e-8)
        assert np.allclose(m.params().astype(np.float64), p - step, rtol=1e-6, atol=1e-5 * lr)
    finally:
        m.close()
