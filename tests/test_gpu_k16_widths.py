"""The 16-bit exchange at column counts on both sides of the line between its GEMM1 tiles
(the 416-column tile padding 30% more than the others, 609 to 640 columns, and 33%,
577 to 608): every tile forms the same products in the same order, so K is bitwise that of
any forced tile, and within the bound of rounding C and X once of the FP64 oracle's K of
the rounded B (u = 2^-8, 2^-11; 2 u each of the sum of absolute values)."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host, system

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("td,u", [(torch.bfloat16, 2.0 ** -8), (torch.float16, 2.0 ** -11)])
@pytest.mark.parametrize("ncol", [417, 576, 609, 624, 625, 640])
def test_widths(ncol, td, u):
    import paper_2506_06661_amd as pkg
    from paper_2506_06661_amd import dfjk
    nao, naux = 640, 3
    print(f"16-bit K, {ncol} columns, {td}", flush=True)
    _, B, _ = system(nao, naux, 1, seed=81)
    C = np.linalg.qr(np.random.default_rng(ncol).standard_normal((nao, ncol)))[0]
    Bq = dev(B, td)
    o = dfjk.default_options()
    o.k16 = 1
    h = pkg.Handle(Bq, nao, opts=o)
    K = host(h.K(C=dev(C)))
    for tile in (0, 1, 4, 7):
        dfjk.dfjk_set_tile(h.h, dfjk.DFJK_TILE_K16, tile)
        assert np.array_equal(host(h.K(C=dev(C))), K), tile
    h.close()
    B64 = host(Bq.double())
    ref = oracle.K_C(B64, nao, C)
    scale = oracle.K_D(np.abs(B64), nao, 2 * np.abs(C) @ np.abs(C).T)
    assert np.all(np.abs(K - ref) <= 4 * u * scale)
