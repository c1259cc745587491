"""Exchange at the edges of the half-transform's and the contraction's tile
forms: nao and column counts around 16, 64, 112, 128 and 144, odd column counts
(the FP64 copy of C), factors meeting inside a 16-row chunk, and calls of fewer
columns than reserved.

Bounds: every K entry is a sum of products x y, x and y sums of nao products
each, added up in at most R + 2 roundings, so the error is below
(2 nao + R + 8) u times the same sums of magnitudes, K(|B|, |C|); R = naux ncol
terms.  u = 2^-53, or 2^-24 for FP32 B (C rounded to FP32 is one of the 8).
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host, system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("nao", [1, 15, 17, 64, 111, 113, 127, 128, 129, 145, 241, 257])
def test_K_tile_edges(nao, dtype):
    import paper_2506_06661_amd as pkg
    naux = 21
    R, B, _ = system(nao, naux, 1, nao)
    if dtype == "f32":
        B = B.astype(np.float32).astype(np.float64)
    Bd = dev(B) if dtype == "f64" else dev(B, torch.float32)
    u = 2.0 ** -53 if dtype == "f64" else 2.0 ** -24
    rng = np.random.default_rng(nao)
    h = pkg.Handle(Bd, nao)
    for ncol in sorted({1, 3, 16, 17, min(nao, 66), min(nao, 113), nao}):
        if ncol > nao:
            continue
        print(f"K edges {dtype} nao={nao} ncol={ncol}", flush=True)
        C = rng.standard_normal((nao, ncol))
        bound = (2 * nao + naux * ncol + 8) * u * oracle.K_C(np.abs(B), nao, np.abs(C))
        assert np.all(np.abs(host(h.K(C=dev(C))) - oracle.K_C(B, nao, C)) <= bound)
        # the two factors of a symmetric pair: 2 naux ncol terms, meeting at naux ncol
        L, Rf = C, rng.standard_normal((nao, ncol))
        D = L @ Rf.T + Rf @ L.T
        Da = np.abs(L) @ np.abs(Rf).T
        bound = (2 * nao + 2 * naux * ncol + 8) * u * oracle.K_D(np.abs(B), nao, Da + Da.T)
        assert np.all(np.abs(host(h.K_pair(dev(L), dev(Rf), sym=True)) - oracle.K_D(B, nao, D)) <= bound)
    h.close()


@pytest.mark.parametrize("max_ncol,ncols", [(41, (40, 41, 39, 1)), (48, (48, 33, 17))])
def test_reserved_fewer_columns(max_ncol, ncols):
    """600 x 40 rows are cut into more splits than 600 x 41: both are reserved."""
    import paper_2506_06661_amd as pkg
    from paper_2506_06661_amd import dfjk
    nao, naux = 64, 600
    R, B, _ = system(nao, naux, 1, 5)
    o = dfjk.default_options()
    o.max_ncol = max_ncol
    Bd = dev(B)
    h, free = pkg.Handle(Bd, nao, opts=o), pkg.Handle(Bd, nao)
    for ncol in ncols:
        print(f"reserved {max_ncol}, used {ncol}", flush=True)
        C = dev(np.random.default_rng(ncol).standard_normal((nao, ncol)))
        assert torch.equal(h.K(C=C), free.K(C=C))
    h.close()
    free.close()
