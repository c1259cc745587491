"""The eigensolver on matrices whose squares leave the range of double: a power of two
is exact, so the eigenvectors of 2^p F are those of F and hold to the bound of
the sweeps (off-diagonal norm 1e-13 of the norm, about 10 sweeps that round every
entry n times by 3 u), for every form of the eigensolver.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("p", [-1010, -570, -401, 399, 520, 1010])
@pytest.mark.parametrize("n", [2, 40, 140, 170, 205])
def test_scaled(n, p):
    import paper_2506_06661_amd as pkg
    print(f"eigenvectors of 2^{p} F, n={n}", flush=True)
    F = np.random.default_rng(n).standard_normal((n, n))
    F = F + F.T
    F.flat[0] = 8.0  # no entry above, so 2^1010 F is far from overflow
    F = np.clip(F, -8.0, 8.0)
    B = torch.zeros((1, n * (n + 1) // 2), dtype=torch.float64, device="cuda")
    h = pkg.Handle(B, n)
    C = torch.zeros((n, n), dtype=torch.float64, device="cuda")
    pkg.dfjk_aufbau(h.h, dev(np.ldexp(F, p)), n, C, None)
    C = host(C)
    h.close()
    tol = 1e-13 + 30 * n * 2.0 ** -53
    w = np.linalg.eigvalsh(F)
    assert np.abs(C.T @ C - np.eye(n)).max() <= tol * np.sqrt(n)
    assert np.abs(C.T @ F @ C - np.diag(w)).max() <= tol * np.linalg.norm(F)


@pytest.mark.parametrize("p", [-560, 500])
@pytest.mark.parametrize("n", [20, 201])
def test_scaled_eigenvalues(n, p):
    """K of a density on a reserved handle: columns sqrt|w| v, so K(2^p D) = 2^p K(D),
    with the sweeps' bound for w and v and n naux FP64 terms summed in both."""
    import paper_2506_06661_amd as pkg
    print(f"K of 2^{p} D, n={n}", flush=True)
    rng = np.random.default_rng(n)
    o = pkg.dfjk.default_options()
    o.max_ncol = n
    h = pkg.Handle(dev(rng.standard_normal((3, n * (n + 1) // 2))), n, opts=o)
    D = rng.standard_normal((n, n))
    D = D + D.T
    K = host(h.K(D=dev(D)))
    Ks = host(h.K(D=dev(np.ldexp(D, p))))
    h.close()
    tol = 10 * (1e-13 + 30 * n * 2.0 ** -53) * np.sqrt(n)
    assert np.abs(np.ldexp(Ks, -p) - K).max() <= tol * np.abs(K).max()
