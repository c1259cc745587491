"""The work that programs built on this library have it do, as cases to time.

Each case is a dict of plain values; ``prepare`` makes what such a program
holds before the call (B, orbitals, densities, handles, batches, network
parameters, all on the GPU), ``run`` makes one pass through the public entry
points, ``work`` counts the bytes and operations a pass cannot do without and
``exact`` gives the same outputs in 64 bits from plain torch.

Kinds:

* ``jk``        J(D) and K(C_occ) of one molecule: the two calls of every SCF
                iteration.  B in FP64, FP32, BF16 or FP16; ``k16`` runs the
                exchange of 16-bit B on the 16-bit matrix cores.
* ``density``   J(D) and K(D) for a density without orbitals (a learned or
                superposed guess: the first build of an SCF).
* ``response``  J of several densities and K of a two-factor density plus its
                transpose (second-order SCF trial vectors).
* ``scf``       the first iterations of an SCF from the core guess, the record
                read after each one as a driver does.
* ``batch``     J and K of many molecules of uneven size, replayed from the
                recorded graph.
* ``batch_scf`` the first SCF iterations of many molecules at once.
* ``train``     training steps of the guess network (loss, gradient, Adam) and
                the parameters read back, as a training loop saves them.
* ``predict``   pair features and network output for one molecule.
* ``form_b``    B = L^-1 Q from the auxiliary metric and the 3-index integrals.

Inputs follow the library's synthetic workloads: basis functions on a cubic
lattice of 1.5 bohr, B[P, mu nu] = a_P exp(-|R_mu - R_nu|^2 / 2) z with
a_P ~ U(0.1, 1), z ~ N(0, 1); orthonormal occupied orbitals; for SCF the core
Hamiltonian -diag(U(1, 5)) + 0.1 exp(-r^2) N(0, 1) and B scaled by 0.005.
"""
import math

import numpy as np
import torch

import paper_2506_06661_amd as pkg
from paper_2506_06661_amd import dfjk, guess

DEV = "cuda"
F64 = torch.float64
CODES = {"f64": pkg.DFJK_F64, "f32": pkg.DFJK_F32, "bf16": pkg.DFJK_BF16, "f16": pkg.DFJK_F16}
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
SIZE = {"f64": 8, "f32": 4, "bf16": 2, "f16": 2}
SCF_SCALE = 0.005
HIDDEN, D_IN = 256, 8


def listed():
    return [
        # the smallest molecule a program builds J and K for: launches and latency
        {"name": "jk_f64_64", "kind": "jk", "dtype": "f64", "k16": False, "nao": 64, "naux": 256, "nocc": 16},
        # 50-100 atoms in FP64: the library's headline workload
        {"name": "jk_f64_1024", "kind": "jk", "dtype": "f64", "k16": False, "nao": 1024, "naux": 4096, "nocc": 200},
        # a mid-size molecule of odd sizes, B stored in single precision
        {"name": "jk_f32_701", "kind": "jk", "dtype": "f32", "k16": False, "nao": 701, "naux": 2803, "nocc": 139},
        # the largest: nao=2048 with 16-bit B and the 16-bit exchange
        {"name": "jk_bf16_k16_2048", "kind": "jk", "dtype": "bf16", "k16": True, "nao": 2048, "naux": 4096,
         "nocc": 400},
        # the first build of an SCF that starts from a density without orbitals
        {"name": "density_f64_400", "kind": "density", "dtype": "f64", "nao": 400, "naux": 1600, "nocc": 80},
        # a second-order SCF step: J of several trial densities, K of one
        {"name": "response_f64_500", "kind": "response", "nao": 500, "naux": 2000, "nocc": 96, "ndm": 6},
        # the SCF family: six iterations from the core guess
        {"name": "scf_f64_128", "kind": "scf", "nao": 128, "naux": 512, "nocc": 24, "iters": 6},
        # many molecules, one graph replay; FP32 B
        {"name": "batch_f32_64", "kind": "batch", "dtype": "f32", "k16": False, "nmol": 64, "lo": 40, "hi": 400,
         "sizes": 4},
        # the same with 16-bit B and the 16-bit exchange
        {"name": "batch_bf16_k16_64", "kind": "batch", "dtype": "bf16", "k16": True, "nmol": 64, "lo": 40,
         "hi": 400, "sizes": 5},
        # SCF iterations of many small molecules at once
        {"name": "batch_scf_16", "kind": "batch_scf", "nmol": 16, "lo": 40, "hi": 160, "sizes": 6, "iters": 3},
        # four training steps of the guess network at the training batch size
        {"name": "train_f32_65536", "kind": "train", "compute": "f32", "rows": 65536, "steps": 4},
        # the 3-index factor of a mid-size molecule
        {"name": "form_b_1536", "kind": "form_b", "naux": 1536, "nao": 384},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["jk", "jk", "jk", "density", "response", "scf", "batch", "batch_scf", "train", "predict",
                       "form_b"])
    if kind == "jk":
        dtype = rng.choice(["f64", "f64", "f32", "bf16", "f16"])
        nao = _log(rng, 48, 1024 if SIZE[dtype] > 2 else 1500)
        return {"kind": kind, "dtype": dtype, "k16": SIZE[dtype] == 2 and rng.random() < 0.6, "nao": nao,
                "naux": int(nao * rng.uniform(2.0, 4.0)), "nocc": max(1, int(nao * rng.uniform(0.08, 0.25)))}
    if kind == "density":
        nao = _log(rng, 40, 480)
        return {"kind": kind, "dtype": rng.choice(["f64", "f64", "f32"]), "nao": nao,
                "naux": int(nao * rng.uniform(1.0, 4.0)), "nocc": max(1, nao // 5)}
    if kind == "response":
        nao = _log(rng, 48, 600)
        return {"kind": kind, "nao": nao, "naux": int(nao * rng.uniform(2.0, 4.0)),
                "nocc": max(1, int(nao * rng.uniform(0.08, 0.25))), "ndm": rng.randint(2, 10)}
    if kind == "scf":
        nao = rng.randint(24, 160)
        return {"kind": kind, "nao": nao, "naux": 4 * nao, "nocc": max(1, nao // 5), "iters": rng.randint(3, 6)}
    if kind == "batch":
        dtype = rng.choice(["f32", "bf16", "f16"])
        return {"kind": kind, "dtype": dtype, "k16": SIZE[dtype] == 2 and rng.random() < 0.6,
                "nmol": _log(rng, 8, 64), "lo": rng.randint(30, 60), "hi": rng.randint(120, 400),
                "sizes": rng.randrange(1 << 20)}
    if kind == "batch_scf":
        return {"kind": kind, "nmol": rng.randint(4, 16), "lo": rng.randint(24, 60), "hi": rng.randint(90, 160),
                "sizes": rng.randrange(1 << 20), "iters": rng.randint(2, 3)}
    if kind == "train":
        return {"kind": kind, "compute": rng.choice(["f32", "bf16"]), "rows": _log(rng, 2000, 65536),
                "steps": rng.randint(2, 4)}
    if kind == "predict":
        return {"kind": kind, "compute": rng.choice(["f32", "bf16"]), "nao": _log(rng, 40, 400)}
    return {"kind": "form_b", "naux": _log(rng, 60, 1536), "nao": _log(rng, 24, 384)}


# ------------------------------------------------------------------ inputs
def _npair(nao):
    return nao * (nao + 1) // 2


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _positions(nao):
    n = int(math.ceil(nao ** (1 / 3) - 1e-9))
    ax = 1.5 * torch.arange(n, device=DEV, dtype=F64)
    x, y, z = torch.meshgrid(ax, ax, ax, indexing="ij")
    return torch.stack([x.reshape(-1), y.reshape(-1), z.reshape(-1)], 1)[:nao].contiguous()


def _r2(R):
    return ((R[:, None, :] - R[None, :, :]) ** 2).sum(-1)


def _pairs(nao):
    return torch.tril_indices(nao, nao, device=DEV)


def _B(R, naux, dtype, g, scale=1.0):
    """Packed B (naux x npair) in its storage type, made in blocks of rows."""
    nao = R.shape[0]
    i, j = _pairs(nao)
    np_ = i.numel()
    # numbers are drawn in the storage width or in FP32, whichever is wider
    wide = F64 if dtype == "f64" else torch.float32
    decay = torch.exp(-0.5 * _r2(R))[i, j].to(wide) * scale
    a = 0.1 + 0.9 * torch.rand(naux, 1, generator=g, device=DEV, dtype=wide)
    B = torch.empty((naux, np_), dtype=TORCH[dtype], device=DEV)
    step = max(1, min(naux, (1 << 28) // np_))
    for p in range(0, naux, step):
        q = min(naux, p + step)
        B[p:q] = torch.randn(q - p, np_, generator=g, device=DEV, dtype=wide).mul_(decay).mul_(a[p:q])
    return B


def _orth(nao, ncol, seed, salt):
    g = torch.Generator()
    g.manual_seed(int(seed) * 7919 + salt)
    return torch.linalg.qr(torch.randn(nao, ncol, generator=g, dtype=F64))[0].contiguous().to(DEV)


def _hamiltonian(R, g):
    nao = R.shape[0]
    H = torch.randn(nao, nao, generator=g, device=DEV, dtype=F64)
    H = 0.1 * torch.exp(-_r2(R)) * (H + H.T) / math.sqrt(2.0)
    H -= torch.diag(1.0 + 4.0 * torch.rand(nao, generator=g, device=DEV, dtype=F64))
    return H.contiguous()


def _sizes(case):
    rng = np.random.RandomState(case["sizes"])
    n = rng.randint(case["lo"], case["hi"] + 1, case["nmol"])
    n[0], n[-1] = case["hi"], case["lo"]  # both ends of the range are met
    return [int(x) for x in n]


def _jk_inputs(case, seed):
    R = _positions(case["nao"])
    C = _orth(case["nao"], case["nocc"], seed, 1)
    D = (2.0 * C @ C.T).contiguous()
    return _B(R, case["naux"], case.get("dtype", "f64"), _gen(seed)), C, D


def _density_inputs(case, seed):
    """A density that is no projector: fractional occupations."""
    nao, nocc = case["nao"], case["nocc"]
    R = _positions(nao)
    U = _orth(nao, nao, seed, 2)
    k = torch.arange(nao, device=DEV, dtype=F64)
    occ = 2.0 / (1.0 + torch.exp((k - nocc) / (1.0 + 0.1 * nocc)))
    D = (U * occ) @ U.T
    return _B(R, case["naux"], case["dtype"], _gen(seed)), (0.5 * (D + D.T)).contiguous()


def _response_inputs(case, seed):
    nao, nocc = case["nao"], case["nocc"]
    R = _positions(nao)
    U = _orth(nao, nao, seed, 3)
    C, V = U[:, :nocc].contiguous(), U[:, nocc:]
    g = _gen(seed, 4)
    L = [(V @ (0.1 * torch.randn(nao - nocc, nocc, generator=g, device=DEV, dtype=F64))).contiguous()
         for _ in range(case["ndm"])]
    D = torch.stack([l @ C.T + C @ l.T for l in L]).contiguous()
    return _B(R, case["naux"], "f64", _gen(seed)), L[0], C, D


def _scf_inputs(nao, naux, seed, dtype):
    R = _positions(nao)
    g = _gen(seed, 5)
    R = (R + 0.1 * torch.randn(nao, 3, generator=g, device=DEV, dtype=F64)).contiguous()
    return _B(R, naux, dtype, g, SCF_SCALE), _hamiltonian(R, g)


def _batch_inputs(case, seed):
    out = []
    for k, nao in enumerate(_sizes(case)):
        nocc = max(1, nao // 5)
        C = _orth(nao, nocc, seed, 100 + k)
        out.append((_B(_positions(nao), 4 * nao, case["dtype"], _gen(seed, 100 + k)), C, (2.0 * C @ C.T).contiguous()))
    return out


def _places(naos):
    """Where each molecule's matrix begins in one buffer for all (whole
    256-byte pieces), and that buffer's length."""
    at, total = [], 0
    for n in naos:
        at.append(total)
        total += (n * n + 31) // 32 * 32
    return at, total


def _batch_scf_inputs(case, seed):
    return [_scf_inputs(nao, 4 * nao, seed * 131 + k, "f32") + (max(1, nao // 5),)
            for k, nao in enumerate(_sizes(case))]


def _mlp_params(seed):
    """Glorot-uniform weights, zero biases, in the library's flat order."""
    rng = np.random.RandomState(seed % (1 << 31))
    flat = []
    for s in [(HIDDEN, D_IN), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (1, HIDDEN), (1,)]:
        lim = math.sqrt(6.0 / sum(s)) if len(s) == 2 else 0.0
        flat.append(rng.uniform(-1.0, 1.0, int(np.prod(s))) * lim)
    return np.concatenate(flat).astype(np.float32)


def _train_inputs(case, seed):
    """Pair features and density corrections with the family's distributions."""
    n = case["rows"] * case["steps"]
    g = _gen(seed, 6)

    def u(lo, hi):
        return lo + (hi - lo) * torch.rand(n, generator=g, device=DEV)

    def z():
        return torch.randn(n, generator=g, device=DEV)

    r = u(0.0, 12.0)
    e = torch.exp(-0.25 * r * r)
    X = torch.stack([0.3 * e * z(), 0.1 * torch.exp(-r * r) * z(), u(-5.0, -1.0), u(0.0, 4.0), 0.1 * r,
                     torch.exp(-r * r), (r < 0.1).float(), u(0.0, 1.0)], 1).contiguous()
    t = (0.05 * (0.1 + e) * z() + 0.2 * X[:, 0]).contiguous()
    return X, t, _mlp_params(seed)


def _predict_inputs(case, seed):
    nao = case["nao"]
    R = _positions(nao)
    H = _hamiltonian(R, _gen(seed, 7))
    C = _orth(nao, max(1, nao // 5), seed, 8)
    return H, (2.0 * C @ C.T).contiguous(), R, _mlp_params(seed)


def _form_b_inputs(case, seed):
    naux, ncol = case["naux"], _npair(case["nao"])
    g = _gen(seed, 9)
    G = torch.randn(naux, naux, generator=g, device=DEV, dtype=F64)
    M = G @ G.T / naux + 0.05 * torch.eye(naux, device=DEV, dtype=F64)
    Q = _B(_positions(case["nao"]), naux, "f64", g)
    assert Q.shape[1] == ncol
    return (0.5 * (M + M.T)).contiguous(), Q


# ------------------------------------------------------------------ passes
def prepare(case, seed):
    kind = case["kind"]
    if kind == "jk":
        B, C, D = _jk_inputs(case, seed)
        opts = dfjk.default_options()
        opts.k16 = int(case["k16"])
        return {"kind": kind, "h": pkg.Handle(B, case["nao"], opts=opts), "C": C, "D": D}
    if kind == "density":
        B, D = _density_inputs(case, seed)
        return {"kind": kind, "h": pkg.Handle(B, case["nao"]), "D": D}
    if kind == "response":
        B, L, C, D = _response_inputs(case, seed)
        return {"kind": kind, "h": pkg.Handle(B, case["nao"]), "L": L, "C": C, "D": D, "J": torch.empty_like(D)}
    if kind == "scf":
        B, H = _scf_inputs(case["nao"], case["naux"], seed, "f64")
        return {"kind": kind, "h": pkg.Handle(B, case["nao"]), "H": H, "nocc": case["nocc"], "iters": case["iters"]}
    if kind == "batch":
        got = _batch_inputs(case, seed)
        at, total = _places([C.shape[0] for _, C, _ in got])
        J, K = torch.zeros(total, dtype=F64, device=DEV), torch.zeros(total, dtype=F64, device=DEV)
        mols = [{"B": B, "nao": D.shape[0], "C": C, "D": D, "J": J[a:a + D.numel()].view(D.shape),
                 "K": K[a:a + D.numel()].view(D.shape)} for (B, C, D), a in zip(got, at)]
        b = pkg.Batch(mols, CODES[case["dtype"]])
        if case["k16"]:
            b.set_k16(True)
        b.capture()
        return {"kind": kind, "b": b, "J": J, "K": K}
    if kind == "batch_scf":
        mols, Hs = [], []
        for B, H, nocc in _batch_scf_inputs(case, seed):
            nao = H.shape[0]
            mols.append({"B": B, "nao": nao, "C": torch.empty((nao, nocc), dtype=F64, device=DEV),
                         "D": torch.empty_like(H), "J": torch.empty_like(H), "K": torch.empty_like(H)})
            Hs.append(H)
        return {"kind": kind, "b": pkg.Batch(mols, pkg.DFJK_F32), "mols": mols, "H": Hs, "iters": case["iters"]}
    if kind == "train":
        X, t, p = _train_inputs(case, seed)
        m = pkg.MLP(D_IN, HIDDEN, case["rows"])
        m.set_params(p)
        if case["compute"] == "bf16":
            m.set_compute(pkg.DFJK_BF16)
        return {"kind": kind, "m": m, "X": X, "t": t, "rows": case["rows"], "steps": case["steps"],
                "loss": torch.zeros(case["steps"], device=DEV)}
    if kind == "predict":
        H, D, R, p = _predict_inputs(case, seed)
        m = pkg.MLP(D_IN, HIDDEN, _npair(case["nao"]))
        m.set_params(p)
        if case["compute"] == "bf16":
            m.set_compute(pkg.DFJK_BF16)
        return {"kind": kind, "m": m, "H": H, "D": D, "R": R}
    M, Q = _form_b_inputs(case, seed)
    return {"kind": kind, "M": M, "Q": Q}


def _record(info):
    return [info.e_tot, info.e_1e, info.e_j, info.e_k]


def run(s):
    kind = s["kind"]
    if kind == "jk":
        return {"J": s["h"].J(s["D"]), "K": s["h"].K(C=s["C"])}
    if kind == "density":
        return {"J": s["h"].J(s["D"]), "K": s["h"].K(D=s["D"])}
    if kind == "response":
        dfjk.dfjk_build_J_multi(s["h"].h, s["D"].shape[0], s["D"], s["J"])
        return {"J": s["J"], "K": s["h"].K_pair(s["L"], s["C"], sym=True)}
    if kind == "scf":
        # The density is returned for the orbitals: single columns of C are
        # defined only up to sign and rotations among near-degenerate levels.
        h, H, nocc = s["h"], s["H"], s["nocc"]
        dfjk.dfjk_scf_reset(h.h)
        C, D = guess.core_guess(h, H, nocc)
        recs = []
        for _ in range(s["iters"]):
            _, info = dfjk.dfjk_scf_step(h.h, H, D, C, nocc, dfjk.DFJK_SCF_C_VALID)
            recs.append(_record(info))
        return {"E": torch.tensor(recs, dtype=F64), "D": D}
    if kind == "batch":
        s["b"].launch()
        return {"J": s["J"], "K": s["K"]}
    if kind == "batch_scf":
        s["b"].scf_guess(s["H"])
        recs = []
        for _ in range(s["iters"]):
            _, info = s["b"].scf_step(s["H"])
            recs.append([_record(i) for i in info])
        return {"E": torch.tensor(recs, dtype=F64), "D": [m["D"] for m in s["mols"]]}
    if kind == "train":
        m, n = s["m"], s["rows"]
        for k in range(s["steps"]):
            m.loss_grad(s["X"][k * n:(k + 1) * n], s["t"][k * n:(k + 1) * n], s["loss"][k:k + 1])
            m.adam(1e-3)
        return {"loss": s["loss"], "params": m.params()}
    if kind == "predict":
        X = guess.features(s["H"], s["D"], s["R"])
        y = torch.empty(X.shape[0], device=DEV)
        s["m"].forward(X, y)
        return {"X": X, "y": y}
    M, Q = s["M"].clone(), s["Q"].clone()  # the call works in place
    pkg.dfjk_form_B(M.shape[0], Q.shape[1], M, Q, Q.shape[1])
    return {"L": M, "B": Q}


# ------------------------------------------------------------------ work
def _k_flops(naux, nao, ncol):
    return 2.0 * naux * nao * nao * ncol + 1.0 * naux * ncol * nao * (nao + 1)


def work(case):
    kind = case["kind"]
    if kind in ("jk", "density", "response", "scf"):
        nao, naux, nocc = case["nao"], case["naux"], case["nocc"]
        b = SIZE[case.get("dtype", "f64")] * naux * _npair(nao)
        j = 4.0 * naux * _npair(nao)
        if kind == "jk":
            return {"bytes": b + 8 * (3 * nao * nao + nao * nocc), "flops": j + _k_flops(naux, nao, nocc)}
        if kind == "density":
            return {"bytes": b + 8 * 3 * nao * nao, "flops": j + 2.0 * naux * nao ** 3 + naux * nao * nao * (nao + 1.0)}
        if kind == "response":
            m = case["ndm"]
            return {"bytes": b + 8 * (2 * m * nao * nao + 2 * nao * nocc + nao * nao),
                    "flops": m * j + 4.0 * naux * nao * nao * nocc + 2.0 * naux * nocc * nao * (nao + 1)}
        # an iteration: J, K, the commutator and an eigensolution of order nao^3
        return {"bytes": case["iters"] * (b + 8 * 6 * nao * nao),
                "flops": case["iters"] * (j + _k_flops(naux, nao, nocc) + 12.0 * nao ** 3)}
    if kind == "batch":
        w = [(SIZE[case["dtype"]] * 4 * n * _npair(n) + 8 * (3 * n * n + n * (n // 5)),
              16.0 * n * _npair(n) + _k_flops(4 * n, n, n // 5)) for n in _sizes(case)]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    if kind == "batch_scf":
        it = case["iters"]
        w = [(it * (16 * n * _npair(n) + 48 * n * n),
              it * (16.0 * n * _npair(n) + _k_flops(4 * n, n, max(1, n // 5)) + 12.0 * n ** 3))
             for n in _sizes(case)]
        return {"bytes": sum(x[0] for x in w), "flops": sum(x[1] for x in w)}
    if kind == "train":
        n = case["rows"] * case["steps"]
        return {"bytes": 4 * n * (D_IN + 1) + case["steps"] * 7 * 4 * (HIDDEN * HIDDEN + 12 * HIDDEN),
                "flops": 6.0 * n * (HIDDEN * HIDDEN + (D_IN + 1) * HIDDEN)}
    if kind == "predict":
        n = _npair(case["nao"])
        return {"bytes": 16 * n + 4 * n * (D_IN + 1) + 4 * (HIDDEN * HIDDEN + 11 * HIDDEN),
                "flops": 2.0 * n * (HIDDEN * HIDDEN + (D_IN + 1) * HIDDEN)}
    naux, ncol = case["naux"], _npair(case["nao"])
    return {"bytes": 16 * naux * (naux + ncol), "flops": 1.0 * naux * naux * ncol + naux ** 3 / 3.0}


# ------------------------------------------------------------------ 64 bits
def _dense_blocks(B, nao):
    """(first row, dense FP64 B_P of a block of rows) over all of B."""
    i, j = _pairs(nao)
    at = torch.empty((nao, nao), dtype=torch.int64, device=DEV)
    p = torch.arange(i.numel(), device=DEV)
    at[i, j] = p
    at[j, i] = p
    step = max(1, (1 << 26) // (nao * nao))
    for a in range(0, B.shape[0], step):
        yield a, B[a:a + step].to(F64)[:, at.reshape(-1)].view(-1, nao, nao)


def _jk64(B, nao, Ds, factors):
    """J of each density in Ds and sum of w (B_P L)(B_P R)^T over (w, L, R)."""
    J = [torch.zeros((nao, nao), dtype=F64, device=DEV) for _ in Ds]
    K = torch.zeros((nao, nao), dtype=F64, device=DEV)
    for _, Bd in _dense_blocks(B, nao):
        flat = Bd.reshape(Bd.shape[0], -1)
        for k, D in enumerate(Ds):
            J[k] += (flat.T @ (flat @ D.reshape(-1))).view(nao, nao)
        for w, L, Rf in factors:
            X = (Bd.reshape(-1, nao) @ L).view(-1, nao, L.shape[1]).transpose(1, 2).reshape(-1, nao)
            Y = X if Rf is L else (Bd.reshape(-1, nao) @ Rf).view(-1, nao, L.shape[1]).transpose(1, 2).reshape(-1, nao)
            K += w * (X.T @ Y)
    return J, K


def _aufbau64(F, nocc):
    C = torch.linalg.eigh(F.cpu())[1][:, :nocc].to(DEV).contiguous()
    return C, 2.0 * C @ C.T


def _scf64(B, H, nocc, iters, space=8, max_cond=1e12):
    """SCF iterations from the core guess with Pulay DIIS over the last
    `space` pairs, the oldest dropped for good while the Gram matrix of the
    errors is worse conditioned than max_cond."""
    nao = H.shape[0]
    C, D = _aufbau64(H, nocc)
    Fs, es, recs = [], [], []
    for _ in range(iters):
        J, K = _jk64(B, nao, [D], [(2.0, C, C)])
        F = H + J[0] - 0.5 * K
        e1, ej, ek = (float((D * A).sum()) for A in (H, J[0], K))
        recs.append([e1 + 0.5 * ej - 0.25 * ek, e1, 0.5 * ej, -0.25 * ek])
        Fs.append(F)
        es.append((F @ D - D @ F))
        Fs, es = Fs[-space:], es[-space:]
        while len(es) > 1:
            E = torch.stack([e.reshape(-1) for e in es])
            w = torch.linalg.eigvalsh((E @ E.T).cpu())
            if w[0] > 0 and w[-1] / w[0] <= max_cond:
                break
            Fs, es = Fs[1:], es[1:]
        m = len(es)
        E = torch.stack([e.reshape(-1) for e in es])
        A = torch.zeros((m + 1, m + 1), dtype=F64)
        A[:m, :m] = (E @ E.T).cpu()
        A[:m, m] = A[m, :m] = -1.0
        rhs = torch.zeros(m + 1, dtype=F64)
        rhs[m] = -1.0
        c = torch.linalg.solve(A, rhs)[:m]
        C, D = _aufbau64(sum(float(ci) * Fi for ci, Fi in zip(c, Fs)), nocc)
    return recs, D


def _unflatten(p):
    out, o = [], 0
    for s in [(HIDDEN, D_IN), (HIDDEN,), (HIDDEN, HIDDEN), (HIDDEN,), (1, HIDDEN), (1,)]:
        n = int(np.prod(s))
        out.append(p[o:o + n].view(s))
        o += n
    return out


def _net64(p, X):
    W1, b1, W2, b2, W3, b3 = _unflatten(p)
    h = torch.nn.functional.silu(X @ W1.T + b1)
    h = torch.nn.functional.silu(h @ W2.T + b2)
    return (h @ W3.T + b3)[:, 0]


def exact(case, seed):
    kind = case["kind"]
    if kind == "jk":
        B, C, D = _jk_inputs(case, seed)
        J, K = _jk64(B, case["nao"], [D], [(2.0, C, C)])
        return {"J": J[0], "K": K}
    if kind == "density":
        B, D = _density_inputs(case, seed)
        eye = torch.eye(case["nao"], dtype=F64, device=DEV)
        J, K = _jk64(B, case["nao"], [D], [(1.0, D, eye)])
        return {"J": J[0], "K": K}
    if kind == "response":
        B, L, C, D = _response_inputs(case, seed)
        J, K = _jk64(B, case["nao"], list(D), [(1.0, L, C)])
        return {"J": torch.stack(J), "K": K + K.T}
    if kind == "scf":
        B, H = _scf_inputs(case["nao"], case["naux"], seed, "f64")
        recs, D = _scf64(B, H, case["nocc"], case["iters"])
        return {"E": torch.tensor(recs, dtype=F64), "D": D}
    if kind == "batch":
        got = _batch_inputs(case, seed)
        at, total = _places([C.shape[0] for _, C, _ in got])
        J, K = torch.zeros(total, dtype=F64, device=DEV), torch.zeros(total, dtype=F64, device=DEV)
        for (B, C, D), a in zip(got, at):
            j, k = _jk64(B, C.shape[0], [D], [(2.0, C, C)])
            J[a:a + D.numel()], K[a:a + D.numel()] = j[0].reshape(-1), k.reshape(-1)
        return {"J": J, "K": K}
    if kind == "batch_scf":
        got = [_scf64(B, H, nocc, case["iters"]) for B, H, nocc in _batch_scf_inputs(case, seed)]
        recs = torch.tensor([r for r, _ in got], dtype=F64).transpose(0, 1).contiguous()
        return {"E": recs, "D": [D for _, D in got]}
    if kind == "train":
        X, t, p0 = _train_inputs(case, seed)
        p = torch.from_numpy(p0).to(DEV, F64)
        m, v = torch.zeros_like(p), torch.zeros_like(p)
        b1, b2, loss = 0.9, 0.999, []
        n = case["rows"]
        for k in range(case["steps"]):
            p.requires_grad_(True)
            L = ((_net64(p, X[k * n:(k + 1) * n].to(F64)) - t[k * n:(k + 1) * n].to(F64)) ** 2).mean()
            g, = torch.autograd.grad(L, p)
            loss.append(float(L.detach()))
            m = b1 * m + (1 - b1) * g
            v = b2 * v + (1 - b2) * g * g
            p = (p - 1e-3 * (m / (1 - b1 ** (k + 1))) / (torch.sqrt(v / (1 - b2 ** (k + 1))) + 1e-8)).detach()
        return {"loss": torch.tensor(loss, dtype=F64), "params": p}
    if kind == "predict":
        H, D, R, p = _predict_inputs(case, seed)
        i, j = _pairs(case["nao"])
        d = torch.diagonal(H)
        rank = torch.argsort(torch.argsort(d, stable=True), stable=True).to(F64)
        r2 = _r2(R)[i, j]
        X = torch.stack([D[j, i], H[j, i], 0.5 * (d[i] + d[j]), (d[i] - d[j]).abs(), 0.1 * torch.sqrt(r2),
                         torch.exp(-r2), (i == j).to(F64), (rank[i] + rank[j]) * 0.5 / case["nao"]], 1)
        return {"X": X, "y": _net64(torch.from_numpy(p).to(DEV, F64), X)}
    M, Q = _form_b_inputs(case, seed)
    L = torch.linalg.cholesky(M.cpu())
    inv = torch.linalg.solve_triangular(L, torch.eye(case["naux"], dtype=F64), upper=False).to(DEV)
    # one correction step: B <- B + L^-1 (Q - L B)
    L = L.to(DEV)
    B = inv @ Q
    return {"L": L, "B": B + inv @ (Q - L @ B)}
