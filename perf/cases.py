"""The purification workloads that this repository is timed on.

Every case is work that a user's program has the library do through its public
entry points: a solve with a kept context (a self-consistency loop, which
purifies a new Hamiltonian of the same size at every step), a one-shot solve,
the solve without allocation, a solve with its gradient, and the FP64
acceptance checks.  The precisions are those that reach the paper's accuracy
(FP64, FP32, FP16X3, BF16X6) and a schedule of two of them.  FP64 solves return
float64 density matrices; the others, which carry 22 to 24 bits, float32.

``exact`` is the closed form: the projector onto the N lowest eigenvectors,
its Daleckii-Krein derivative, and the definitions of the acceptance checks.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1512_07236_amd as gcp

DEVICE = "cuda"
F64 = torch.float64


# ------------------------------------------------------------------- the cases
def _case(name, kind, matrix, M, N, precision, **more):
    c = {"kind": kind, "matrix": matrix, "M": M, "N": N, "gap": 0.0, "precision": precision,
         "late": "", "bwd": "", "method": "hpcp", "init": "pmcp", "gershgorin": False,
         "tol_ddbar": 1e-6, "tol_idem": 0.0}
    if name:
        c["name"] = name
    c.update(more)
    return c


def listed():
    return [
        # the open chain of 256 sites, to FP64 idempotency: the smallest solve,
        # where launches and host checks count
        _case("chain_256_fp64", "solve", "chain", 256, 100, "fp64", tol_ddbar=0.0, tol_idem=1e-10),
        # the quick start: one call, bounds from the Gershgorin discs, nothing kept
        _case("oneshot_520_fp64", "oneshot", "spectral", 520, 200, "fp64", gap=0.1,
              gershgorin=True),
        # the solve that allocates nothing, for serving loops; a ragged size
        _case("static_777_fp16x3", "static", "spectral", 777, 300, "fp16x3", gap=0.1),
        # a low filling, where the alpha search saves a third of the updates
        _case("search_1500_fp16x3", "solve", "spectral", 1500, 75, "fp16x3", gap=0.1,
              init="search"),
        # the 16 x 16 x 8 lattice with the gradient of a loss, through autograd
        _case("lattice_2048_autograd", "autograd", "lattice", 2048, 682, "fp64", bwd="fp64",
              tol_ddbar=1e-8),
        # a mixed start finished in FP64, for tolerances below the mixed floor
        _case("schedule_2048", "solve", "spectral", 2048, 800, "fp16x3", gap=0.1, late="fp64",
              tol_ddbar=1e-9),
        # 24-bit products at an ordinary, ragged size
        _case("ragged_2500_bf16x6", "solve", "spectral", 2500, 1000, "bf16x6", gap=0.1),
        # FP64 acceptance checks of a mixed-precision result
        _case("verify_3000", "verify", "spectral", 3000, 1200, "fp64", gap=0.1),
        # single precision just below a round size
        _case("ragged_3900_fp32", "solve", "spectral", 3900, 1950, "fp32", gap=0.1),
        # the dense FP64 workload
        _case("spectral_4096_fp64", "solve", "spectral", 4096, 2048, "fp64", gap=0.1,
              tol_ddbar=1e-9),
        # a mixed solve and its FP32 gradient, in a training loop
        _case("gradient_4096", "gradient", "spectral", 4096, 1600, "fp16x3", gap=0.2, bwd="fp32"),
        # the headline workload: M = 8192, N = 3000, gap 0.05
        _case("spectral_8192_fp16x3", "solve", "spectral", 8192, 3000, "fp16x3", gap=0.05),
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["solve", "solve", "solve", "solve", "low", "oneshot", "static", "schedule",
                       "gradient", "autograd", "verify"])
    gap = round(rng.uniform(0.05, 0.3), 3)
    theta = rng.uniform(0.2, 0.8)
    if kind == "solve":
        prec = rng.choice(["fp64", "fp32", "fp16x3", "fp16x3", "bf16x6"])
        M = size(100, 8192 if prec == "fp16x3" else 6000)
        return _case("", "solve", "spectral", M, int(theta * M), prec, gap=gap,
                     method=rng.choice(["hpcp", "hpcp", "pmcp"]))
    if kind == "low":
        M = size(200, 5000)
        return _case("", "solve", "spectral", M, max(2, int(rng.uniform(0.03, 0.15) * M)),
                     rng.choice(["fp64", "fp16x3"]), gap=gap, init="search")
    if kind == "oneshot":
        M = size(100, 4000)
        return _case("", "oneshot", "spectral", M, int(theta * M), rng.choice(["fp64", "fp16x3"]),
                     gap=gap, gershgorin=True)
    if kind == "static":
        M = size(64, 1024)
        return _case("", "static", "spectral", M, int(theta * M),
                     rng.choice(["fp64", "fp16x3", "bf16x6"]), gap=gap)
    if kind == "schedule":
        M = size(300, 4096)
        return _case("", "solve", "spectral", M, int(theta * M), rng.choice(["fp16x3", "bf16x6"]),
                     gap=gap, late="fp64", tol_ddbar=1e-9)
    if kind == "gradient":
        M = size(200, 4096)
        return _case("", "gradient", "spectral", M, int(rng.uniform(0.3, 0.7) * M), "fp16x3",
                     gap=round(rng.uniform(0.2, 0.4), 3), bwd="fp32")
    if kind == "autograd":
        M = size(100, 2500)
        return _case("", "autograd", "spectral", M, int(theta * M), "fp64", gap=gap, bwd="fp64",
                     tol_ddbar=1e-8)
    M = size(100, 4096)
    return _case("", "verify", "spectral", M, int(theta * M), "fp64", gap=gap)


# ------------------------------------------------------------------ the inputs
def _spectral(case, seed):
    """H = Q diag(lam) Q^T with N eigenvalues in [-1, -gap/2] and the others in
    [gap/2, 1].  Q = S1 C S2 C with random signs S and the orthogonal cosine
    matrix C: dense, with entries close to Gaussian, without a QR."""
    M, N, gap = case["M"], case["N"], case["gap"]
    rng = np.random.default_rng(seed)
    lam = np.concatenate([rng.uniform(-1.0, -gap / 2, N), rng.uniform(gap / 2, 1.0, M - N)])
    s1, s2 = rng.choice([-1.0, 1.0], M), rng.choice([-1.0, 1.0], M)
    perm = rng.permutation(M)
    k = 2 * torch.arange(M, device=DEVICE) + 1
    C = (k[:, None] * k[None, :]) % (8 * M)
    C = torch.cos(C.to(F64) * (math.pi / (4 * M))) * math.sqrt(2.0 / M)
    Q = torch.as_tensor(s1, device=DEVICE)[:, None] * (C @ (torch.as_tensor(s2, device=DEVICE)[:, None] * C))
    Q = Q[:, torch.as_tensor(perm, device=DEVICE)].contiguous()
    lam = torch.as_tensor(lam, device=DEVICE)
    H = (Q * lam) @ Q.T
    return 0.5 * (H + H.T), Q, lam, (-1.0, 1.0)


def _chain(case, seed):
    M = case["M"]
    rng = np.random.default_rng(seed)
    H = np.zeros((M, M))
    H[np.diag_indices(M)] = rng.uniform(-0.5, 0.5, M)
    i = np.arange(M - 1)
    H[i, i + 1] = H[i + 1, i] = -1.0
    return torch.as_tensor(H, device=DEVICE), None, None, (-2.5, 2.5)


def _lattice(case, seed):
    """Periodic 16 x 16 x (M / 256) simple-cubic lattice, hopping -1."""
    M = case["M"]
    L = (16, 16, M // 256)
    rng = np.random.default_rng(seed)
    H = np.zeros((M, M))
    H[np.diag_indices(M)] = rng.uniform(-1.0, 1.0, M)
    s = np.arange(M)
    x, y, z = s % 16, (s // 16) % 16, s // 256
    for dx, dy, dz in ((1, 0, 0), (0, 1, 0), (0, 0, 1)):
        t = (x + dx) % L[0] + 16 * ((y + dy) % L[1]) + 256 * ((z + dz) % L[2])
        np.add.at(H, (s, t), -1.0)
        np.add.at(H, (t, s), -1.0)
    return torch.as_tensor(H, device=DEVICE), None, None, (-7.0, 7.0)


def _problem(case, seed):
    return {"spectral": _spectral, "chain": _chain, "lattice": _lattice}[case["matrix"]](case, seed)


def _eigen(case, seed):
    """Occupied and empty eigenvectors and eigenvalues, with H."""
    H, Q, lam, _ = _problem(case, seed)
    N = case["N"]
    if Q is None:
        lam, Q = torch.linalg.eigh(H)
    return H, Q[:, :N], Q[:, N:], lam[:N], lam[N:]


def _loss_gradient(case, seed):
    """dL/dD of L = Tr(D P), P symmetric with Gaussian entries."""
    g = torch.Generator(device=DEVICE).manual_seed(seed + 77)
    P = torch.randn((case["M"], case["M"]), generator=g, device=DEVICE, dtype=F64)
    P = 0.5 * (P + P.T)
    return P if case["kind"] == "autograd" else P.to(torch.float32)


def _checked_matrix(case, seed, Qo):
    """A projector with the symmetric error of a mixed-precision solve."""
    g = torch.Generator(device=DEVICE).manual_seed(seed + 99)
    M = case["M"]
    E = torch.randn((M, M), generator=g, device=DEVICE, dtype=F64)
    return Qo @ Qo.T + (E + E.T) * (3e-7 / math.sqrt(M))


def _dtype(case):
    return F64 if case["precision"] == "fp64" else torch.float32


def prepare(case, seed):
    H, Q, _, (emin, emax) = _problem(case, seed)
    M, N, kind = case["M"], case["N"], case["kind"]
    if case["gershgorin"]:
        emin = emax = math.nan
    state = {"kind": kind, "H": H, "N": N, "emin": emin, "emax": emax, "precision": case["precision"],
             "dtype": _dtype(case)}
    options = {"tol_ddbar": case["tol_ddbar"], "tol_idem": case["tol_idem"]}
    if kind == "static":
        state["options"] = options
        state["D"] = torch.empty((M, M), dtype=_dtype(case), device=DEVICE)
        return state
    options.update(method=case["method"], init=case["init"], precision=case["precision"])
    if case["late"]:
        options.update(late_precision=case["late"], switch_ddbar=1e-2)
    if kind in ("gradient", "autograd"):
        options["bwd_precision"] = case["bwd"]
        state["G"] = _loss_gradient(case, seed)
    if kind in ("oneshot", "autograd"):
        state["options"] = options
        if kind == "autograd":
            state["H"] = H.requires_grad_()
        return state
    state["ctx"] = gcp.Context(M, keep_iterates=kind == "gradient", **options)
    if kind == "verify":
        state["D"] = _checked_matrix(case, seed, Q[:, :N])
    else:
        state["D"] = torch.empty((M, M), dtype=_dtype(case), device=DEVICE)
    return state


# -------------------------------------------------------------------- one pass
def run(state):
    kind, H, N, lo, hi = (state[k] for k in ("kind", "H", "N", "emin", "emax"))
    if kind == "static":
        D, _, _ = gcp.purify_static(H, N, lo, hi, out=state["D"], precision=state["precision"],
                                    **state["options"])
        return D
    if kind == "oneshot":
        D, _ = gcp.purify(H, N, lo, hi, out=torch.empty_like(H, dtype=state["dtype"]),
                          **state["options"])
        return D
    if kind == "autograd":
        D = gcp.purify_autograd(H, N, lo, hi, **state["options"])
        dH, = torch.autograd.grad(D, H, state["G"])
        return {"D": D, "dH": dH}
    ctx = state["ctx"]
    if kind == "verify":
        r = ctx.verify(state["D"], H)
        return {k: r[k] for k in ("trace", "fro2", "idem", "energy", "comm")}
    ctx.init(H, N, lo, hi)
    D, _ = ctx.purify(out=state["D"])
    if kind == "gradient":
        dH, _ = ctx.backward(state["G"])
        return {"D": D, "dH": dH}
    return D


# ------------------------------------------------------------------ the measure
def _updates(case):
    """Updates that the recursion takes (its eigenvalue map, on an even
    spectrum; the chain and the lattice take 20 and 26)."""
    if case["matrix"] != "spectral":
        return 20 if case["matrix"] == "chain" else 26
    M, N, gap = case["M"], case["N"], case["gap"]
    lam = np.concatenate([np.linspace(-1.0, -gap / 2, N), np.linspace(gap / 2, 1.0, M - N)])
    theta, mu = N / M, lam.mean()
    r = 0.46 * math.sqrt(M) if case["gershgorin"] else 1.0   # half width of the bounds
    beta = min(theta / (r - mu), (1 - theta) / (mu + r))
    if case["init"] == "search":
        beta = math.sqrt(max(N / 3 - N * theta, 0.05 * N) / ((lam - mu) ** 2).sum())
    x = theta + beta * (mu - lam)
    for p in range(100):
        t1, t2, t3 = x.sum(), (x * x).sum(), (x ** 3).sum()
        if abs(t1 - t2) <= max(case["tol_ddbar"], 1e-12):
            return p
        c = (t2 - t3) / (t1 - t2)
        x = x + 2 * (x * x * (1 - x) - c * x * (1 - x))
    return 100


def work(case):
    M, kind = case["M"], case["kind"]
    sym, gen = float(M) * M * (M + 1), 2.0 * M ** 3
    out = 8 if case["precision"] == "fp64" else 4
    if kind == "verify":
        return {"bytes": 16 * M * M, "flops": sym + gen}
    p = _updates(case)
    flops, size = 2 * p * sym, (8 + out) * M * M
    if kind in ("gradient", "autograd"):
        g = 8 if kind == "autograd" else 4
        flops += p * (2 * sym + 2 * gen)
        size += 2 * g * M * M
    return {"bytes": size, "flops": flops}


def exact(case, seed):
    H, Qo, Qv, lo, lv = _eigen(case, seed)
    kind = case["kind"]
    if kind == "verify":
        D = _checked_matrix(case, seed, Qo)
        X = H @ D
        return {"trace": float(D.trace()), "fro2": float((D * D).sum()),
                "idem": float(torch.linalg.norm(D @ D - D)), "energy": float((D * H).sum()),
                "comm": float(torch.linalg.norm(X - X.T))}
    D = Qo @ Qo.T
    if kind not in ("gradient", "autograd"):
        return D
    # Daleckii-Krein: the occupied-empty block of the loss gradient, divided by
    # the eigenvalue differences
    F = (Qo.T @ _loss_gradient(case, seed).to(F64) @ Qv) / (lo[:, None] - lv[None, :])
    dH = Qo @ F @ Qv.T
    return {"D": D, "dH": dH + dH.T}
