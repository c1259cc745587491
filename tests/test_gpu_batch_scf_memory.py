"""Device memory and results of SCF steps over more molecules than one launch holds
(64): beyond (8 + 2 * 8) nao^2 doubles a molecule only 64 logs of 40 nao^2 doubles, and
every molecule as if it were alone.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def molecules(sizes, rng):
    mols, H = [], []
    for n in sizes:
        a = rng.standard_normal((n, n))
        H.append(dev(0.05 * (a + a.T) - np.diag(rng.uniform(1.0, 5.0, n))))
        B = dev(0.005 * rng.standard_normal((4, synth.npair(n))), torch.float32)
        mols.append({"B": B, "nao": n, "C": torch.zeros((n, max(1, n // 5)), dtype=torch.float64, device="cuda"),
                     **{k: torch.zeros((n, n), dtype=torch.float64, device="cuda") for k in "DJK"}})
    return mols, H


def test_memory():
    import paper_2506_06661_amd as pkg
    n, nmol = 198, 160
    mols, H = molecules([n] * nmol, np.random.default_rng(1))
    b = pkg.Batch(mols, pkg.DFJK_F32)
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    print(f"guess of {nmol} molecules of {n}", flush=True)
    b.scf_guess(H)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    b.close()
    # allocations come in whole 2 MiB; 64 MiB for kernels loaded on first use
    bound = nmol * (24 * 8 * n * n + (4 << 20)) + 64 * 40 * 8 * n * n + (64 << 20)
    assert used <= bound, (used, bound)


def test_shared_logs():
    import paper_2506_06661_amd as pkg
    rng = np.random.default_rng(2)
    sizes = [int(x) for x in rng.integers(3, 60, 150)] + [90, 140, 5]
    mols, H = molecules(sizes, rng)
    keep = [{k: m[k].clone() for k in "DCJK"} for m in mols]
    print("three steps of all molecules", flush=True)
    b = pkg.Batch(mols, pkg.DFJK_F32)
    b.scf_guess(H)
    e = [[i.e_tot for i in b.scf_step(H)[1]] for _ in range(3)]
    b.close()
    for i in (0, 63, 64, 100, 127, 128, 149, 150, 151, 152):
        one = {**mols[i], **keep[i]}
        b = pkg.Batch([one], pkg.DFJK_F32)
        b.scf_guess([H[i]])
        for k in range(3):
            assert b.scf_step([H[i]])[1][0].e_tot == e[k][i], (i, k)
        assert np.array_equal(host(one["D"]), host(mols[i]["D"])) and np.array_equal(host(one["C"]), host(mols[i]["C"]))
        b.close()
