"""The network's kernels at the edges of their tiles, against the FP64 oracle:
hidden widths around 64 (registers per lane), 128 (tile) and 256 (row passes),
odd widths and d_in that is no multiple of 8, batches around the row blocks
(16), the weight-gradient slab (512) and one past them.

Bound per gradient block: every entry is a chain of FP32 sums over the hidden
units and over the batch; with the probabilistic bound of Higham & Mary (2019),
lambda = 10, its error is below (10 (sqrt(H) + sqrt(n)) + 40) u times the same
gradient computed with absolute values (u = 2^-24; 40 u for the elementwise
steps and the exponential).
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

CASES = [(8, 256, 1), (8, 256, 17), (8, 256, 513), (1, 16, 130), (9, 17, 255), (20, 100, 129), (8, 130, 1025),
         (64, 257, 64), (3, 300, 511), (8, 1024, 40)]


def abs_grad(params, X, t):
    """The loss gradient's sums with every term taken by absolute value."""
    W1, b1, W2, b2, W3, b3 = [np.abs(p) for p in params]
    _, (Xs, z1, h1, z2, h2) = oracle.mlp_forward(params, X)
    y = np.abs(h2) @ W3.T + b3
    gy = (2.0 / X.shape[0]) * (y + np.abs(t)[:, None])
    h1, h2, X = np.abs(h1), np.abs(h2), np.abs(X)
    gz2 = (gy @ W3) * 1.1          # |silu'| < 1.1
    gz1 = (gz2 @ W2) * 1.1
    return y[:, 0], [gz1.T @ X, gz1.sum(0), gz2.T @ h1, gz2.sum(0), gy.T @ h2, gy.sum(0)]


@pytest.mark.parametrize("d_in,hidden,n", CASES)
def test_network_edges(d_in, hidden, n):
    import torch
    import paper_2506_06661_amd as pkg
    print(f"network d_in={d_in} hidden={hidden} n={n}", flush=True)
    m = pkg.MLP(d_in=d_in, hidden=hidden, max_batch=n)
    flat = (0.6 * synth.normal(31, synth.STREAM_MLP, m.nparam) / np.sqrt(hidden)).astype(np.float32)
    m.set_params(flat)
    params = [p.astype(np.float64) for p in m.unflatten(flat)]
    X = synth.normal(32, synth.STREAM_MLP, n * d_in).reshape(n, d_in).astype(np.float32)
    t = synth.normal(33, synth.STREAM_MLP, n).astype(np.float32)
    Xd, td = dev(X, torch.float32), dev(t, torch.float32)
    y = torch.empty(n, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    m.forward(Xd, y)
    m.loss_grad(Xd, td, loss)
    u = 2.0 ** -24
    bound = (10 * (np.sqrt(hidden) + np.sqrt(n)) + 40) * u
    X64, t64 = X.astype(np.float64), t.astype(np.float64)
    y_ref, _ = oracle.mlp_forward(params, X64)
    y_abs, g_abs = abs_grad(params, X64, t64)
    L_ref, g_ref = oracle.mlp_loss_grad(params, X64, t64)
    assert np.all(np.abs(host(y) - y_ref) <= bound * y_abs)
    assert abs(float(host(loss)[0]) - L_ref) <= bound * float(np.mean((y_abs + np.abs(t64)) ** 2))
    for k, (a, b, s) in enumerate(zip(m.unflatten(m.grads()), g_ref, g_abs)):
        err = np.abs(a.reshape(b.shape) - b)
        assert np.all(err <= bound * s.reshape(b.shape)), (k, float(err.max()))
    g1 = m.grads()
    m.loss_grad(Xd, td, loss)
    assert np.array_equal(g1, m.grads())  # reproducible
    m.close()
