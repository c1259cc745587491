"""Sums of the training step over the largest batch, 2^24 rows.  All rows are
equal, so the loss and its gradient are those of one row, and the roundings of a
running sum of equal terms all go one way: the worst case for a long FP32 chain.
"""
import numpy as np
import pytest

from gpu_util import host

pytestmark = pytest.mark.gpu
ROWS = 1 << 24
U = 2.0 ** -24


def step(params, x, t):
    """Loss and flat gradient of ROWS rows x with target t, hidden width 16."""
    import torch
    import paper_2506_06661_amd as pkg
    m = pkg.MLP(d_in=1, hidden=16, max_batch=ROWS)
    m.set_params(np.concatenate([p.ravel() for p in params]).astype(np.float32))
    X = torch.full((ROWS, 1), x, dtype=torch.float32, device="cuda")
    T = torch.full((ROWS,), t, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    m.loss_grad(X, T, loss)
    out = float(host(loss)[0]), m.unflatten(m.grads())
    m.close()
    return out


@pytest.mark.parametrize("t", [0.1, 1.0 / 3.0])
def test_loss(t):
    """Output weights 0: y = 0, every square is t^2 exactly in FP64.  Rounded are a
    wavefront's sum, three additions of the workgroup and the result: 5 u; 8 u allowed
    (a chain of 256 FP32 partial sums alone can be 128 u off)."""
    print(f"loss of {ROWS} rows, t={t}", flush=True)
    params = [np.ones((16, 1)), np.zeros(16), np.eye(16), np.zeros(16), np.zeros((1, 16)), np.zeros(1)]
    loss, _ = step(params, 0.5, t)
    ref = float(np.float32(t)) ** 2
    assert abs(loss - ref) <= 8 * U * ref


def test_gradient():
    """No FP32 running sum is longer than 2048 rows in the hidden weights' gradient
    and 4096 in the others (a wavefront's rows); their partials are added in FP64.  64 u
    more for the elementwise steps, relative to the sums of absolute values."""
    import oracle
    print(f"gradient of {ROWS} rows", flush=True)
    rng = np.random.default_rng(5)
    params = [rng.uniform(0.1, 1.0, s).astype(np.float32) for s in ((16, 1), 16, (16, 16), 16, (1, 16), 1)]
    x, t = 0.7, 0.3
    p64 = [p.astype(np.float64) for p in params]
    # one row; every weight and activation is positive, so no sum cancels
    L, g = oracle.mlp_loss_grad(p64, np.array([[float(np.float32(x))]]), np.array([float(np.float32(t))]))
    loss, got = step(params, x, t)
    for k, (a, b) in enumerate(zip(got, g)):
        rel = np.abs(a.reshape(b.shape) - b) / np.abs(b)
        print(k, rel.max() / U, flush=True)
        assert rel.max() <= ((2048 if k == 2 else 4096) + 64) * U, (k, rel.max() / U)
    assert abs(loss - L) <= 200 * U * L
