"""Norms of the eigenvectors, in 80 bits.  A rotation's c^2 + s^2 errs by about u, to
either side; over the rounds of 10 sweeps the mean of |v|^2 - 1 over the n vectors is a
random walk of 10 n steps of size u sqrt(2 / n) (n / 2 rotations each): sqrt(20) u.  Ten
times that is allowed; an error to one side would add up to n u and more.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [60, 86, 130, 198])
def test_norms(n):
    import paper_2506_06661_amd as pkg
    print(f"norms of eigenvectors, n={n}", flush=True)
    F = np.random.default_rng(n).standard_normal((n, n))
    h = pkg.Handle(torch.zeros((1, n * (n + 1) // 2), dtype=torch.float64, device="cuda"), n)
    C = torch.empty((n, n), dtype=torch.float64, device="cuda")
    pkg.dfjk_aufbau(h.h, dev(F + F.T), n, C, None)
    v = host(C).astype(np.longdouble)
    h.close()
    drift = float(((v * v).sum(0) - 1).mean())
    print(drift, flush=True)
    assert abs(drift) <= 10 * np.sqrt(20) * 2.0 ** -53
