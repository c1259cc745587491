"""FP64 dense kernels at the edges of their forms: the factor B = L^-1 Q around
the 64-row blocks and 256-row panels of the substitution and the 64 columns of a
workgroup, and the commutator of one SCF step on both sides of the small
product's largest result (640).

Bounds: B as in the other tests of this entry point (1e-10 of the largest entry;
condition numbers below 1e3).  Commutator with B = 0, so F = H: each entry is two
sums of n products, an error of at most 2 n u |H|_F |D|_F in all, doubled for
the summed squares and the root.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import dev, host, max_rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("naux,ncol", [(63, 1), (65, 64), (255, 65), (256, 63), (257, 128), (320, 17), (513, 129),
                                       (577, 66)])
def test_form_B_edges(naux, ncol):
    import paper_2506_06661_amd as pkg
    print(f"form_B naux={naux} ncol={ncol}", flush=True)
    M = synth.metric(naux, naux)
    Q = np.random.default_rng(naux).standard_normal((naux, ncol + 1))
    Mu = M.copy()
    Mu[np.triu_indices(naux, 64)] = np.nan  # blocks above the diagonal's are not read
    Mu[np.tril_indices(naux, 0)] = M[np.tril_indices(naux, 0)]
    Md, Qd = dev(Mu), dev(Q)
    pkg.dfjk_form_B(naux, ncol, Md, Qd, ncol + 1)
    B = host(Qd)
    assert max_rel(B[:, :ncol], oracle.form_B(M, Q[:, :ncol])) < 1e-10
    assert np.array_equal(B[:, ncol], Q[:, ncol])
    L = host(Md)
    assert max_rel(L, np.linalg.cholesky(M)) < 1e-12
    assert np.all(np.triu(L, 1) == 0)


@pytest.mark.parametrize("nao", [1, 15, 17, 64, 97, 449, 641])
def test_scf_commutator(nao):
    import paper_2506_06661_amd as pkg
    print(f"commutator nao={nao}", flush=True)
    rng = np.random.default_rng(nao)
    H = rng.standard_normal((nao, nao))
    H = H + H.T
    nocc = max(1, nao // 3)
    C = np.linalg.qr(rng.standard_normal((nao, nocc)))[0]
    D = 2 * C @ C.T
    B = torch.zeros((1, nao * (nao + 1) // 2), dtype=torch.float64, device="cuda")
    h = pkg.Handle(B, nao)
    Dd, Cd = dev(D), dev(C)
    rc, info = pkg.dfjk_scf_step(h.h, dev(H), Dd, Cd, nocc, pkg.DFJK_SCF_C_VALID)
    e = np.linalg.norm(H @ D - D @ H)
    bound = 4 * nao * 2.0 ** -53 * np.linalg.norm(H) * np.linalg.norm(D)
    assert abs(info.err_norm - e) <= bound
    Cn = host(Cd)
    assert np.abs(host(Dd) - 2 * Cn @ Cn.T).max() <= 8 * nocc * 2.0 ** -53
    h.close()
