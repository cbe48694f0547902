"""The warm start's gradient and Adam steps at batch sizes around the eighths that the waves of
the reduction take (fewer samples than waves, remainders, whole eighths), against FP64 numpy:
gradients and loss to 1e-5 of the largest entry, as the oracle tests of the gradient."""
import numpy as np
import pytest

from paper_2408_16509_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [1, 7, 8, 9, 63, 64, 257, 1000])
def test_gradient_and_training_at_batch_sizes(n):
    from paper_2408_16509_amd import frmi
    ctx = frmi.Context(inputs.hex_box((2, 2, 2)), order=1)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, 16)).astype(np.float32)
    y = rng.uniform(size=n).astype(np.float32)
    w = inputs.mlp_glorot(5)
    mean, std = np.zeros(16), np.ones(16)
    ctx.mlp_set_weights(w, mean, std)
    X, Y = torch.tensor(x, device="cuda"), torch.tensor(y, device="cuda")
    g, loss = ctx.mlp_grad(X, Y)

    def grad64(wf):
        W1, b1 = wf[:1024].reshape(64, 16), wf[1024:1088]
        W2, b2 = wf[1088:5184].reshape(64, 64), wf[5184:5248]
        w3, b3 = wf[5248:5312], wf[5312]
        h1 = np.tanh(x.astype(np.float64) @ W1.T + b1)
        h2 = np.tanh(h1 @ W2.T + b2)
        r = h2 @ w3 + b3 - y
        dy = 2 * r / n
        d2 = dy[:, None] * w3 * (1 - h2 ** 2)
        d1 = (d2 @ W2) * (1 - h1 ** 2)
        return np.concatenate([(d1.T @ x).ravel(), d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0), dy @ h2,
                               [dy.sum()]]), np.mean(r ** 2)
    want, l64 = grad64(w.astype(np.float64))
    assert abs(float(loss) - l64) <= 1e-5 * l64
    assert np.abs(g.cpu().numpy() - want).max() <= 1e-5 * np.abs(want).max()
    # three Adam steps on the whole set
    wf, mm, vv = w.astype(np.float64), 0.0, 0.0
    for t in range(1, 4):
        gr, _ = grad64(wf)
        mm, vv = 0.9 * mm + 0.1 * gr, 0.999 * vv + 0.001 * gr * gr
        wf = wf - 1e-3 * (mm / (1 - 0.9 ** t)) / (np.sqrt(vv / (1 - 0.999 ** t)) + 1e-8)
    rows = torch.arange(n, dtype=torch.int32, device="cuda").repeat(3)
    ctx.mlp_train(X, Y, rows, 3, n)
    # an Adam step is lr times a ratio of O(1): entries whose gradient is rounding alone may
    # move by it, so the bound is on the norm
    got = ctx.mlp_get_weights()
    assert np.linalg.norm(got - wf) <= 1e-2 * np.linalg.norm(wf - w)
    ctx.close()
