"""Signed columns in GEMM2 and two-factor densities in FP32, at column counts around
the 16-row chunk (a row's column is carried from chunk to chunk: fewer columns than
rows, one more, one less), odd contraction lengths and one to several output tiles, against
the FP64 oracle.

Bound: sums over nao (GEMM1) and naux x columns (GEMM2) terms; with the probabilistic
bound of Higham & Mary (2019), lambda = 10, the error is below (10 (sqrt(nao) +
sqrt(naux columns)) + 40) u times the sum of absolute values.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host, system

pytestmark = pytest.mark.gpu


def setup(nao, naux, ncol, dtype):
    import paper_2506_06661_amd as pkg
    _, B, _ = system(nao, naux, 1, seed=61)
    if dtype == torch.float32:
        B = B.astype(np.float32).astype(np.float64)
    C = np.random.default_rng(ncol).standard_normal((nao, ncol))
    u = 2.0 ** -53 if dtype == torch.float64 else 2.0 ** -24
    return pkg, pkg.Handle(dev(B, dtype), nao), B, C, (10 * (np.sqrt(nao) + np.sqrt(naux * ncol)) + 40) * u


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nao,naux,ncol", [(20, 37, 1), (20, 37, 3), (40, 61, 15), (40, 61, 16), (130, 101, 17),
                                           (150, 55, 33), (90, 700, 7)])
def test_signs(nao, naux, ncol, dtype):
    print(f"signs nao={nao} naux={naux} ncol={ncol} {dtype}", flush=True)
    pkg, h, B, C, bound = setup(nao, naux, ncol, dtype)
    sign = np.where(np.random.default_rng(ncol + 1).random(ncol) < 0.5, -1.0, 1.0)
    K = torch.empty((nao, nao), dtype=torch.float64, device="cuda")
    pkg.dfjk_build_K_factored(h.h, dev(C), ncol, dev(sign), 0.75, K)
    ref = oracle.K_D(B, nao, 0.75 * (C * sign) @ C.T)
    scale = oracle.K_D(np.abs(B), nao, 0.75 * np.abs(C) @ np.abs(C).T)
    h.close()
    assert np.all(np.abs(host(K) - ref) <= bound * scale)


@pytest.mark.parametrize("nao,naux,ncol", [(20, 37, 1), (130, 101, 17), (300, 40, 5)])
def test_pairs(nao, naux, ncol):
    print(f"pairs nao={nao} naux={naux} ncol={ncol}", flush=True)
    pkg, h, B, C, bound = setup(nao, naux, ncol, torch.float32)
    R = np.random.default_rng(ncol + 2).standard_normal((nao, ncol))
    D, A = C @ R.T, np.abs(C) @ np.abs(R).T
    K = host(h.K_pair(dev(C), dev(R), True))
    h.close()
    ref, scale = oracle.K_D(B, nao, D + D.T), oracle.K_D(np.abs(B), nao, A + A.T)
    assert np.all(np.abs(K - ref) <= bound * scale)
