"""Matrices with an infinity or a NaN: no eigenvectors exist, so every value that
dfjk_aufbau, the batched guess and the eigen-factors of a density write is NaN,
whatever the outputs held before, and nothing beside them is written.  One size per
form of the eigensolver (one and three blocks per thread, one copy in LDS, global
memory), the entry on and off the diagonal.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host

pytestmark = pytest.mark.gpu

BAD = [((0, 0), np.nan), ((-1, -1), np.inf), ((0, -1), np.nan), ((-1, 0), -np.inf)]


def handle(n, max_ncol=0):
    import paper_2506_06661_amd as pkg
    o = pkg.dfjk.default_options()
    o.max_ncol = max_ncol
    B = torch.zeros((1, n * (n + 1) // 2), dtype=torch.float64, device="cuda")
    return pkg.Handle(B, n, opts=o)


def guarded(*shape):
    """A tensor of ones inside a longer buffer, and a check that the rest stays as it was."""
    n = int(np.prod(shape))
    buf = torch.ones(n + 128, dtype=torch.float64, device="cuda")
    return buf[64:64 + n].view(shape), lambda: bool((host(buf)[:64] == 1).all() and (host(buf)[-64:] == 1).all())


@pytest.mark.parametrize("n", [1, 2, 90, 140, 198, 199, 230])
def test_aufbau(n):
    import paper_2506_06661_amd as pkg
    F0 = np.random.default_rng(n).standard_normal((n, n))
    h = handle(n)
    for at, value in BAD:
        print(f"aufbau n={n} {value} at {at}", flush=True)
        F = F0.copy()
        F[at] = value
        nocc = max(1, n // 2)
        (C, keptC), (D, keptD) = guarded(n, nocc), guarded(n, n)
        pkg.dfjk_aufbau(h.h, dev(F), nocc, C, D)
        assert np.isnan(host(C)).all() and np.isnan(host(D)).all()
        assert keptC() and keptD()
    # the handle still solves a finite matrix
    C = torch.empty((n, n), dtype=torch.float64, device="cuda")
    pkg.dfjk_aufbau(h.h, dev(F0), n, C, None)
    assert np.abs(host(C).T @ host(C) - np.eye(n)).max() <= 1e-10
    h.close()


@pytest.mark.parametrize("n", [60, 210])
def test_density_factors(n):
    """K of a density on a reserved handle goes through the eigen-factors of D."""
    h = handle(n, max_ncol=n)
    D = np.eye(n)
    D[1, 2] = D[2, 1] = np.nan
    print(f"K of a density with a NaN, n={n}", flush=True)
    assert np.isnan(host(h.K(D=dev(D)))).all()
    h.close()


def test_batch_guess():
    """One bad molecule leaves the others as they would be without it."""
    import paper_2506_06661_amd as pkg
    sizes = [30, 90, 140]
    rng = np.random.default_rng(3)
    H = [(lambda a: a + a.T)(rng.standard_normal((n, n))) for n in sizes]
    out = []
    for bad in (False, True):
        if bad:
            H[1][4, 7] = np.nan
        mols = [{"B": torch.zeros((1, n * (n + 1) // 2), dtype=torch.float32, device="cuda"), "nao": n,
                 "C": torch.ones((n, n // 3), dtype=torch.float64, device="cuda"),
                 **{k: torch.ones((n, n), dtype=torch.float64, device="cuda") for k in "DJK"}} for n in sizes]
        b = pkg.Batch(mols, pkg.DFJK_F32)
        print(f"batch guess, NaN: {bad}", flush=True)
        b.scf_guess([dev(x) for x in H])
        out.append([host(m["D"]) for m in mols])
        b.close()
    assert np.isnan(out[1][1]).all()
    for i in (0, 2):
        assert np.isfinite(out[0][i]).all() and np.array_equal(out[0][i], out[1][i])
