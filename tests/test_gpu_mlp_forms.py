"""Fused gradient step of the quadrature network at the edges of its chunks.

Batches of one sample, one chunk (16 samples), one more, several workgroups
with a ragged last chunk, and more chunks than workgroups (256 x 16), against
the FP64 oracle's chain rule; a training run whose batches end ragged against
the same steps taken one gradient at a time.  Tolerance 1e-5 of the largest
entry: FP32 sums of up to a few thousand terms of mixed sign, whose rounding
grows like a random walk, sqrt(4113) x 2^-24 = 4e-6.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _data(n, seed):
    rng = np.random.default_rng(seed)
    nt = rng.choice([6, 8, 10, 12], size=n)
    X = np.stack([rng.uniform(-3, 0, n), rng.uniform(0.25, 1, n), nt / 12.0], 1).astype(np.float32)
    M = np.tile(np.arange(12)[None, :] < nt[:, None], 2).astype(np.float32)
    Y = (rng.standard_normal((n, 24)) * 2.0 - 1.0).astype(np.float32) * M
    return X, Y, M


@pytest.fixture(scope="module")
def L():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1611_06797_amd import ltmp2
    return ltmp2


@pytest.mark.parametrize("n", [1, 15, 16, 17, 1023, 4096, 4113])
def test_gradient_chunks_vs_oracle(L, n):
    from oracle import mlp
    print("[gpu-case] mlp gradient, batch", n, flush=True)
    X, Y, M = _data(n, n)
    p = L.mlp_init(3)
    g, loss = L.mlp_grad(p, X, Y, M)
    ref = mlp.grad(p.astype(np.float64), X, Y, M)
    assert abs(loss - mlp.loss(p.astype(np.float64), X, Y, M)) <= 1e-5 * loss
    assert np.abs(g - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("n,batch", [(40, 13), (33, 16), (5, 9)])
def test_training_steps_are_adam_on_the_gradient(L, n, batch):
    print("[gpu-case] mlp training", n, batch, flush=True)
    X, Y, M = _data(n, 7)
    p = L.mlp_init(1)
    hist = L.mlp_train(p, X, Y, M, 1, batch, 1e-2, 11)
    # the library's epoch order: Fisher-Yates with splitmix64
    s, mask = 11, (1 << 64) - 1

    def uniform():
        nonlocal s
        s = (s + 0x9E3779B97F4A7C15) & mask
        z = s
        z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & mask
        z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & mask
        return ((z ^ (z >> 31)) >> 11) * 2.0 ** -53
    perm = list(range(n))
    for k in range(n - 1, 0, -1):
        q = int(uniform() * (k + 1))
        perm[k], perm[q] = perm[q], perm[k]
    batch = min(batch, n)
    from oracle import mlp
    r = L.mlp_init(1).astype(np.float64)
    m = v = np.zeros_like(r)
    loss = cnt = 0.0
    for step, b0 in enumerate(range(0, n - batch + 1, batch), 1):
        k = perm[b0:b0 + batch]
        g = mlp.grad(r, X[k], Y[k], M[k])
        loss += mlp.loss(r, X[k], Y[k], M[k]) * M[k].sum()
        cnt += M[k].sum()
        m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
        r = r - 1e-2 * (m / (1 - 0.9 ** step)) / (np.sqrt(v / (1 - 0.999 ** step)) + 1e-8)
    assert abs(hist[0] - loss / cnt) <= 1e-5 * hist[0]
    # a step moves every entry by at most 1e-2; entries whose gradient is at
    # rounding level may take the other sign, so the bound is on the mean
    assert np.abs(p - r).mean() <= 1e-5
