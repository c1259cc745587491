"""The network's products in both tile sizes (64 and 128 wide: from 512 tiles of 128 on)
and both compute types at odd widths, one row, remainders of the tiles and of the
contraction's chunks (16 FP32, 32 BF16), against the FP64 oracle.

Bounds: FP32 as in test_gpu_mlp_edges; BF16 adds LAMBDA standard deviations of the
rounded operands (bf16_sigmas).  One training step is also bitwise reproducible.
"""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import dev, host
from test_gpu_mlp import LAMBDA, bf16_sigmas
from test_gpu_mlp_edges import abs_grad

pytestmark = pytest.mark.gpu

# the last two: 172 x 3 and 512 x 1 tiles of 128, the first of them ragged on every side
CASES = [(8, 256, 1), (9, 17, 255), (1, 16, 513), (64, 257, 65), (3, 300, 511), (8, 1024, 40), (5, 257, 21901),
         (2, 33, 65536)]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("d_in,hidden,n", CASES)
def test_network_tiles(d_in, hidden, n, bf16):
    import torch
    import paper_2506_06661_amd as pkg
    print(f"network d_in={d_in} hidden={hidden} n={n} bf16={bf16}", flush=True)
    m = pkg.MLP(d_in=d_in, hidden=hidden, max_batch=n)
    m.set_compute(pkg.DFJK_BF16 if bf16 else pkg.DFJK_F32)
    flat = (0.6 * synth.normal(41, synth.STREAM_MLP, m.nparam) / np.sqrt(hidden)).astype(np.float32)
    m.set_params(flat)
    params = [p.astype(np.float64) for p in m.unflatten(flat)]
    X = synth.normal(42, synth.STREAM_MLP, n * d_in).reshape(n, d_in).astype(np.float32)
    t = synth.normal(43, synth.STREAM_MLP, n).astype(np.float32)
    Xd, td = dev(X, torch.float32), dev(t, torch.float32)
    y = torch.empty(n, dtype=torch.float32, device="cuda")
    loss = torch.empty(1, dtype=torch.float32, device="cuda")
    m.forward(Xd, y)
    m.loss_grad(Xd, td, loss)
    g1 = m.grads()
    m.loss_grad(Xd, td, loss)
    assert np.array_equal(g1, m.grads())
    m.close()
    bound = (10 * (np.sqrt(hidden) + np.sqrt(n)) + 40) * 2.0 ** -24
    X64, t64 = X.astype(np.float64), t.astype(np.float64)
    y_ref, _ = oracle.mlp_forward(params, X64)
    y_abs, g_abs = abs_grad(params, X64, t64)
    _, g_ref = oracle.mlp_loss_grad(params, X64, t64)
    dy, dg = bf16_sigmas(params, X64, t64) if bf16 else (0.0, [0.0] * 6)
    assert np.all(np.abs(host(y) - y_ref) <= bound * y_abs + LAMBDA * dy)
    for k, (a, b, s, d) in enumerate(zip(m.unflatten(g1), g_ref, g_abs, dg)):
        err = np.abs(a.reshape(b.shape) - b)
        assert np.all(err <= bound * s.reshape(b.shape) + LAMBDA * np.reshape(d, b.shape if bf16 else ())), (
            k, float(err.max()))
