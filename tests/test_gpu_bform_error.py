"""Rounding of the 3-index factor against an 80-bit Cholesky and substitution.

Every entry takes one rounding per block of 64 terms (n / 64 of them, each at most u
times the entry) and the sums inside a block, which are a fraction of it: the
root mean square error of L stays below (sqrt(n / 64) + 4) u, with random signs; a rounding
of the whole entry per term would give sqrt(n) u.  The substitution takes over L's
error, and adds its own, by at most the root of L's condition number (9 here):
3 times that bound for B.
"""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def reference(M, Q):
    """Cholesky factor and L^-1 Q in 80 bits, 32 columns at a time."""
    n = M.shape[0]
    L = M.astype(np.longdouble)
    for k in range(0, n, 32):
        e = min(k + 32, n)
        for j in range(k, e):
            L[j, j] = np.sqrt(L[j, j])
            L[j + 1:, j] /= L[j, j]
            L[j + 1:, j + 1:e] -= np.outer(L[j + 1:, j], L[j + 1:e, j])
        for j in range(k, e):
            L[e:, e:] -= np.outer(L[e:, j], L[e:, j])
    L = np.tril(L)
    X = Q.astype(np.longdouble)
    for i in range(n):
        X[i] = (X[i] - L[i, :i] @ X[:i]) / L[i, i]
    return L, X


def rms(x):
    return float(np.sqrt(np.mean(x.astype(np.longdouble) ** 2)))


@pytest.mark.parametrize("naux", [257, 700, 960])
def test_error(naux):
    import paper_2506_06661_amd as pkg
    print(f"form_B error naux={naux}", flush=True)
    rng = np.random.default_rng(naux)
    G = rng.standard_normal((naux, naux))
    M = G @ G.T / naux + 0.05 * np.eye(naux)
    M, Q = 0.5 * (M + M.T), rng.standard_normal((naux, 20))
    Md, Qd = dev(M), dev(Q)
    pkg.dfjk_form_B(naux, 20, Md, Qd, 20)
    L, X = reference(M, Q)
    bound = (np.sqrt(naux / 64) + 4) * 2.0 ** -53
    eL, eB = rms(np.tril(host(Md)) - L) / rms(L), rms(host(Qd) - X) / rms(X)
    print(f"L {eL:.2e} B {eB:.2e} bound {bound:.2e}", flush=True)
    assert eL <= bound and eB <= 3 * bound
