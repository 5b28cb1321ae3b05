"""Training kernels at the edges of their row tiles, chunks and slices: the
gradient against the reference network's, and the z-score statistics against
the same sums in 64 bits, row after row."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 17, 33, 64, 65, 2049, 64 * 65 + 1])
def test_gradient(n):
    import paper_2211_12867_amd as ic
    from oracle import mlp
    g = np.random.default_rng(n)
    p = ic.mlp_init(5).astype(np.float32)
    x = g.standard_normal((n, ic.MLP_IN)).astype(np.float32)
    y = (g.random(n) < 0.3).astype(np.uint8)
    grad, loss = ic.mlp_grad(x, y, p, 2.0)
    rloss, ref = mlp.loss_and_grad(x, y, p, 2.0)
    # rounded at the same points; an fp32 sum that falls on the other side of a rounding point moves a bf16 value
    # by 2^-8 of itself, and a hidden unit whose sum is 0 to rounding drops out or stays: a few parts in 1,000 of a
    # layer's largest entry for one row, less for many
    assert abs(loss - rloss) < 2e-3 * max(1.0, rloss)
    for a, b in ((mlp.OFF_W1, mlp.OFF_B1), (mlp.OFF_B1, mlp.OFF_W2), (mlp.OFF_W2, mlp.OFF_B2),
                 (mlp.OFF_B2, mlp.OFF_W3), (mlp.OFF_W3, mlp.OFF_B3), (mlp.OFF_B3, mlp.OFF_B3 + 1)):
        assert np.abs(grad[a:b] - ref[a:b]).max() < 2e-2 * np.abs(ref[a:b]).max() + 1e-7, (a, b)


@pytest.mark.parametrize("n", [1, 15, 511, 512, 513, 1055])
def test_statistics(n):
    import paper_2211_12867_amd as ic
    g = np.random.default_rng(n)
    raw = (g.standard_normal((n, ic.MLP_IN)) * (1 + np.arange(ic.MLP_IN)) + 7.0).astype(np.float32)
    raw[:, 3] = 2.5                                      # no spread: std 1
    _, mean, std, _ = ic.mlp_train(raw, (np.arange(n) % 2).astype(np.uint8), ic.mlp_init(1), epochs=0, batch=1)
    r = raw.astype(np.float64)
    mu = np.cumsum(r, axis=0)[-1] / n
    sd = np.sqrt(np.cumsum((r - mu) ** 2, axis=0)[-1] / n)
    sd[~(sd > 1e-6)] = 1.0
    assert np.array_equal(mean, mu.astype(np.float32)) and np.array_equal(std, sd.astype(np.float32))
