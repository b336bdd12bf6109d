"""The guess network's kernels at the ends of their passes: 16 rows a
wavefront, 64 a workgroup, FP32 sums flushed after eight passes."""
import numpy as np
import pytest
import torch

from oracle import mlp as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sw():
    import paper_2404_17754_amd as sw
    return sw


def _rows(n, seed):
    rng = np.random.default_rng(seed)
    S = np.zeros((n, 12), np.float32)
    S[:, :10] = rng.uniform(-1, 1, (n, 10))
    S[:, 10] = 0.3 * rng.standard_normal(n)
    S[:, 11] = rng.uniform(0.01, 2.0, n)
    return S


# 256 workgroups of 64 rows: 131072 rows are eight full passes of each
@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 1023, 131072, 140001])
def test_gradient(sw, n):
    th = om.init(3).astype(np.float32)
    rng = np.random.default_rng(4)
    th[4864:] = rng.uniform(-0.3, 0.3, 65)        # a trained-like output layer
    S = _rows(n, n)
    g, loss = sw.Mlp(sw.Context(0), th).gradient(torch.from_numpy(S))
    S64, th64 = S.astype(np.float64), th.astype(np.float64)
    gr = om.gradient(th64, S64[:, :10], S64[:, 10], S64[:, 11])
    # FP32 forward and back: about 100 roundings of 6e-8 deep
    assert np.linalg.norm(g - gr) <= 6e-6 * np.linalg.norm(gr)
    assert abs(loss - om.loss(th64, S64[:, :10], S64[:, 10], S64[:, 11])) <= 6e-6 * loss


def test_training_beyond_the_loss_ring(sw):
    """Losses of more steps than stay on the device at once, and the same
    steps in two calls."""
    S = torch.from_numpy(_rows(500, 1))
    ctx = sw.Context(0)
    a, b = sw.Mlp(ctx, seed=2), sw.Mlp(ctx, seed=2)
    la = a.train(S, steps=1100, batch=20, lr=1e-3, seed=5)
    lb = np.concatenate([b.train(S, steps=1024, batch=20, lr=1e-3, seed=5), b.train(S, steps=76, batch=20, lr=1e-3, seed=5)])
    assert np.all(la > 0) and np.all(np.isfinite(la))
    # the same sums up to their arrival order in FP64
    assert np.abs(la - lb).max() <= 1e-4 * la.max()


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65537 * 16 + 3])
@pytest.mark.parametrize("shift", [0, 1])
def test_forward(sw, n, shift):
    """shift: rows that start at single-value alignment."""
    th = om.init(3).astype(np.float32)
    th[4864:] = np.random.default_rng(4).uniform(-0.3, 0.3, 65)
    X = _rows(n, n + 1)[:, :10]
    buf = torch.zeros(10 * n + 4, device="cuda")
    view = buf[shift:shift + 10 * n].view(n, 10)
    view.copy_(torch.from_numpy(np.ascontiguousarray(X)))
    y = sw.Mlp(sw.Context(0), th).forward(view).cpu().numpy()
    ref = om.forward(th.astype(np.float64), X.astype(np.float64))
    # FP16 inputs, weights and activations: 5e-4 each, of sums over 64 units
    assert np.abs(y - ref).max() <= 8e-3 * np.abs(ref).max()
