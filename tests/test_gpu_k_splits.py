"""The splits of FP64 GEMM2 on both sides of the rule's steps: K against the oracle,
and the partial tiles (their bytes tell the number of splits) at most twice as many, and
one more, where the contraction gets a chunk of 16 rows longer.

Tolerance: sums over nao and naux nocc terms, (10 (sqrt(nao) + sqrt(naux nocc)) + 40) u
(Higham & Mary 2019, lambda = 10) of the sum of absolute values.
"""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host, system

pytestmark = pytest.mark.gpu


def build(nao, naux, nocc):
    """K, its reference and bound, and the bytes of the split partials."""
    import paper_2506_06661_amd as pkg
    _, B, C = system(nao, naux, nocc, seed=71)
    h = pkg.Handle(dev(B), nao)
    before = h.workspace_bytes()
    K = host(h.K(C=dev(C)))
    ldx = (nao + 1) // 2 * 2
    part = h.workspace_bytes() - before - 8 * naux * nocc * ldx
    h.close()
    ref = oracle.K_C(B, nao, C)
    bound = (10 * (np.sqrt(nao) + np.sqrt(naux * nocc)) + 40) * 2.0 ** -53
    scale = oracle.K_D(np.abs(B), nao, 2 * np.abs(C) @ np.abs(C).T)
    assert np.all(np.abs(K - ref) <= bound * scale)
    return part


# contractions of (naux, naux + step) x nocc rows around the steps at 96 rows a split
# within 2 MiB and at 384 rows a split
@pytest.mark.parametrize("nao,naux,nocc,step", [(64, 383, 16, 2), (128, 96, 16, 1), (128, 384, 16, 1), (128, 512, 12, 2),
                                                (112, 480, 16, 1), (200, 160, 12, 2), (200, 30, 16, 1)])
def test_steps(nao, naux, nocc, step):
    print(f"splits nao={nao} naux={naux} nocc={nocc}", flush=True)
    a, b = build(nao, naux, nocc), build(nao, naux + step, nocc)
    slot = (nao + 15) // 16 * 16 if nao < 128 else 128
    nt = (nao + 127) // 128
    one = 8 * slot * slot * (nt * (nt + 1) // 2)
    print(a // one, b // one, "splits", flush=True)
    assert a <= b + one and b <= 2 * a + one
