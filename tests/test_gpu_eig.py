"""The eigensolver through dfjk_aufbau with every orbital asked for, at the
edges of its forms: odd sizes, one and two pairs, one block per thread up to
n = 86, two copies in LDS up to n = 138, one copy up to n = 198, global memory
from 199 on; dense, diagonal, degenerate, zero and non-finite matrices.

Bound: the sweeps stop at an off-diagonal norm of 1e-13 of the matrix norm, and
each of about 10 sweeps rounds every entry n times (3 u per rotation), so
eigenvalues, residuals and orthonormality hold to (1e-13 + 30 n u) |F|_F.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def solve(F):
    import paper_2506_06661_amd as pkg
    n = F.shape[0]
    B = torch.zeros((1, n * (n + 1) // 2), dtype=torch.float64, device="cuda")
    h = pkg.Handle(B, n)
    C = torch.full((n, n), 7.0, dtype=torch.float64, device="cuda")
    D = torch.empty((n, n), dtype=torch.float64, device="cuda")
    pkg.dfjk_aufbau(h.h, dev(F), n, C, D)
    out = host(C), host(D)
    h.close()
    return out


def check(F):
    n = F.shape[0]
    S = 0.5 * (F + F.T)
    C, D = solve(F)
    norm = max(np.linalg.norm(S), 1e-300)
    tol = 1e-13 + 30 * n * 2.0 ** -53
    w = np.linalg.eigvalsh(S)
    assert np.abs(C.T @ C - np.eye(n)).max() <= tol * np.sqrt(n)
    assert np.abs(C.T @ S @ C - np.diag(w)).max() <= tol * norm
    assert np.abs(D - 2 * C @ C.T).max() <= 1e-13 * n


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 86, 87, 128, 129, 138, 139, 197, 198, 199])
def test_dense(n):
    print(f"eig n={n}", flush=True)
    check(np.random.default_rng(n).standard_normal((n, n)))


@pytest.mark.parametrize("n", [6, 87, 140])
def test_special(n):
    print(f"eig special n={n}", flush=True)
    rng = np.random.default_rng(n)
    check(np.zeros((n, n)))
    check(np.diag(rng.standard_normal(n)))
    Q = np.linalg.qr(rng.standard_normal((n, n)))[0]
    check((Q * np.repeat([1.0, -2.0], [n // 2, n - n // 2])) @ Q.T)   # two degenerate levels
    check(1e150 * rng.standard_normal((n, n)))                         # squares overflow: no sweep limit reached


def test_nonfinite_ends(n=90):
    """A NaN must neither hang nor write out of range (values are not defined)."""
    F = np.random.default_rng(1).standard_normal((n, n))
    F[3, 4] = np.nan
    solve(F)
