"""The adjoint at sizes that are not whole tiles, on both sides of half
filling: the rows and columns that pad M to whole tiles may not reach dL/dH.
They would through Tr Gbar_0, whose coefficient in dL/dH vanishes for the
default guess where beta = theta/(emax - mu) (low fillings) and for no other
branch or guess.  Against the oracle's adjoint at the GPU's p; M = 40, 200,
449 and 1000 are padded by 24, 56, 63 and 24 rows.

Tolerances as those of the whole-tile sizes: FP64 1e-12 plus the difference of
the two forwards' c_n, 1e-14 times the purified trace over Tr(D Dbar); FP32
2e-5 per update."""
import numpy as np
import pytest

from oracle import grad
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1512_07236_amd as gcp  # noqa: E402
from test_gpu_adjoint import _oracle, gpu_grad, log, rel_max  # noqa: E402,F401

CASES = [(40, 28, {}), (200, 140, {}), (449, 300, {}), (1000, 700, {}),
         (200, 140, {"method": "pmcp"}),
         (200, 20, {"init": "search"}), (200, 180, {"init": "search"}),
         (200, 120, {"init": "hp", "alpha": 0.5}),
         (200, 60, {"hole": True}), (200, 140, {"hole": True})]


@pytest.mark.parametrize("bwd", ["fp64", "fp32"])
@pytest.mark.parametrize("M,N,opts", CASES)
def test_padding_does_not_reach_the_gradient(M, N, opts, bwd):
    w = workloads.spectral(M, N, 0.2, M + N)
    Gp = workloads.sym_gaussian(M, M + 305)
    dH, res, _ = gpu_grad(w, Gp, bwd_precision=bwd, tol_ddbar=1e-6,
                          dtype=torch.float64 if bwd == "fp64" else torch.float32, **opts)
    p = res.iters
    assert res.status in gcp.SUCCESS
    how = {"method": opts.get("method", "hpcp"), "alpha": opts.get("alpha", 1.0),
           "init": "search" if opts.get("init") == "search" else None}
    ref = grad.adjoint(w.H, N, w.emin, w.emax, p, Gp, **how)
    _, _, t12, _, _ = grad.forward_iterates(w.H, N, w.emin, w.emax, p, **how)
    tol = 2e-5 * p
    if bwd == "fp64":
        tol = 1e-12 + 1e-14 * max(N, M - N if opts.get("hole") else 0) / np.abs(t12).min()
    err = rel_max(dH, ref)
    log(f"  M={M} N={N} {opts} {bwd}: p={p} err={err:.3e} tol={tol:.3e}")
    assert np.array_equal(dH, dH.T)
    assert err <= tol
