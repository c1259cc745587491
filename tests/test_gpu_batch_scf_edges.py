"""Batched SCF at the edges of its launches: molecules on both sides of the
largest matrix the LDS eigensolver takes (198) in one batch, each of its forms,
and more molecules than one launch carries (64), against the single-molecule SCF
on the same FP32 B.

Bound: as for the batched SCF elsewhere: energies agree to the size of the
FP32 sums in E_K, below 1e-6 Eh at this scale of B; the density left behind is
idempotent with trace 2 nocc to 1e-9.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_util import dev

pytestmark = pytest.mark.gpu


def molecule(seed, nao):
    R = synth.cluster_positions(seed, nao)
    B = synth.B_full(seed, R, max(4, 2 * nao)) * synth.C5_B_SCALE
    return B.astype(np.float32), synth.core_hamiltonian(seed, R), max(1, nao // 5)


@pytest.mark.parametrize("naos", [(1, 2, 31, 86, 87, 139, 198), (40, 199, 12, 203), (200,), (9,) * 70])
def test_batch_scf_edges(naos):
    import paper_2506_06661_amd as pkg
    from paper_2506_06661_amd import dfjk
    mols, Hs, singles = [], [], []
    for i, nao in enumerate(naos):
        B, H, nocc = molecule(300 + i, nao)
        print(f"batch scf edge nao={nao} nocc={nocc}", flush=True)
        f64 = dict(dtype=torch.float64, device="cuda")
        mols.append({"B": dev(B, torch.float32), "nao": nao, "D": torch.zeros((nao, nao), **f64),
                     "C": torch.zeros((nao, nocc), **f64), "J": torch.zeros((nao, nao), **f64),
                     "K": torch.zeros((nao, nao), **f64)})
        Hs.append(dev(H))
        h = pkg.Handle(mols[-1]["B"], nao, dtype=dfjk.DFJK_F32)
        C, D = torch.empty((nao, nocc), **f64), torch.empty((nao, nao), **f64)
        dfjk.dfjk_aufbau(h.h, Hs[-1], nocc, C, D)
        dfjk.dfjk_scf_reset(h.h)
        singles.append([dfjk.dfjk_scf_step(h.h, Hs[-1], D, C, nocc, dfjk.DFJK_SCF_C_VALID)[1].e_tot
                        for _ in range(4)])
        h.close()
    b = pkg.Batch(mols, dfjk.DFJK_F32)
    for run in range(2):  # the second starts over in the first one's workspace
        b.scf_guess(Hs)
        for it in range(4):
            _, infos = b.scf_step(Hs)
            for i, inf in enumerate(infos):
                assert inf.iter == it + 1
                assert abs(inf.e_tot - singles[i][it]) < 1e-6, (run, it, i)
    for m in mols:
        D = m["D"].cpu().numpy()
        assert abs(np.trace(D) - 2 * m["C"].shape[1]) < 1e-9 and np.abs(D @ D - 2 * D).max() < 1e-9
    b.close()
