"""The CDF model's gradient kernel (matrix-core blocks of 32 samples, 128 to a
workgroup, at most 256 workgroups) against the fp64 oracle around its block,
workgroup and grid edges, and training run twice.

Tolerance: y is a chain of two 32-term fp32 dot products, so it is off by at
most 80 * 2^-24 of the sum Y of its terms' absolute values, and dy by 2/b times
that.  A gradient entry adds b products of dy with at most 80 further roundings
each, in chains of at most b / 32768 + 1 samples per lane and then 5 + 2 + 16 +
16 partial sums.  With A(d) the sum of the terms' absolute values at dy = d:
|error| <= (80 + 40 + b / 32768) * 2^-24 * A(|dy|) + 80 * 2^-24 * A(2 Y / b),
and 2^-24 times those counts is below 1e-5.
"""
import numpy as np
import pytest
import torch

import paper_2409_03970_amd as hv
from oracle import mlp
from paper_2409_03970_amd import inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _abs_terms(p, x, dy=None, t=None):
    """Sum over the samples of |term| of every gradient entry in fp64, at the
    given dy (or at |dy| of targets t)."""
    W1, b1, W2, b2, W3, b3 = mlp.unpack(p)
    y, (x, z1, h1, z2, h2) = mlp.forward(p, x)
    if dy is None:
        dy = np.abs(2.0 * (y - t) / len(x))
    dz2 = np.outer(dy, np.abs(W3)) * (z2 > 0)
    dz1 = (dz2 @ np.abs(W2)) * (z1 > 0)
    a = np.abs
    return np.concatenate([dz1.T @ a(x), dz1.sum(0), (dz2.T @ a(h1)).reshape(-1), dz2.sum(0),
                           a(h2).T @ dy, [dy.sum()]])


def _abs_y(p, x):
    W1, b1, W2, b2, W3, b3 = (np.abs(v) for v in mlp.unpack(p))
    return (np.outer(np.abs(x), W1) + b1) @ W2.T @ W3 + b2 @ W3 + b3


@pytest.mark.parametrize("b", [1, 31, 32, 33, 127, 128, 129, 4096, 32767, 32768, 32769, 100003])
def test_gradient_at_block_and_grid_edges(b):
    print("gradient", b, flush=True)
    rng = np.random.default_rng(b)
    p = inputs.mlp_init(b).to(DEV)
    x = rng.uniform(0, 1, b).astype(np.float32)
    t = rng.uniform(0, 1, b).astype(np.float32)
    loss, g = hv.cdf_backward(p, torch.from_numpy(x).to(DEV), torch.from_numpy(t).to(DEV))
    pd, xd, td = p.cpu().double().numpy(), x.astype(np.float64), t.astype(np.float64)
    want_loss, want = mlp.backward(pd, xd, td)
    off = _abs_y(pd, xd)
    bound = 1e-5 * (_abs_terms(pd, xd, t=td) + _abs_terms(pd, xd, dy=2 * off / b)) + 1e-12
    err = np.abs(g.cpu().double().numpy() - want)
    assert np.all(err <= bound), (np.argmax(err / bound), (err / bound).max())
    y, _ = mlp.forward(pd, xd)
    assert abs(loss - want_loss) <= 1e-5 * np.mean((y - td) ** 2 + 2 * np.abs(y - td) * off) + 1e-12


@pytest.mark.parametrize("batch", [1, 100, 128, 5000, 32769])
def test_training_is_deterministic(batch):
    """Two runs of three steps are bitwise the same and finite."""
    sample = torch.sort(inputs.keys(10007, "mixture", seed=1, device=DEV)).values
    runs = [hv.cdf_train(inputs.mlp_init(2).to(DEV), sample, batch=batch, steps=k, seed=9)
            for k in (3, 3)]
    for a, c in zip(*runs):
        assert torch.equal(a, c)
    assert all(bool(torch.isfinite(a).all()) for a in runs[0])
