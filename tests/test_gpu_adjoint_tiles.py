"""The adjoint's tile launches at the sizes where their shape changes, against
the oracle's adjoint at the GPU's p: one tile and two tile rows (both products
of every tile split), seven tile rows (28 split tiles), 300 tiles of which 44
are split and 406 of which 150 are, six times each; PMCP, whose kappa needs the D^2 tiles, at seven tile rows."""
import pytest

from oracle import grad
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_adjoint import _oracle, fp64_tol, gpu_grad, log, rel_max  # noqa: E402,F401

SIZES = [(40, 15), (65, 30), (449, 180), (1473, 560), (1750, 700)]


@pytest.mark.parametrize("M,N,method", [(M, N, "hpcp") for M, N in SIZES] + [(449, 180, "pmcp")])
def test_adjoint_at_the_edges(M, N, method):
    w = workloads.spectral(M, N, 0.2, M + 5)
    Gp = workloads.sym_gaussian(M, M + 205)
    opts = {"tol_ddbar": 1e-6, "method": method}
    for prec, dtype in (("fp64", torch.float64), ("fp32", torch.float32)):
        dH, res, bres = gpu_grad(w, Gp, bwd_precision=prec, dtype=dtype, **opts)
        ref = grad.adjoint(w.H, w.N, w.emin, w.emax, res.iters, Gp, method=method)
        err = rel_max(dH, ref)
        tol = fp64_tol(w, res.iters) if prec == "fp64" else 2e-5 * res.iters
        log(f"  M={M} {method} {prec}: p={res.iters} err={err:.3e} tol={tol:.3e}")
        assert bres.iters == res.iters and (dH == dH.T).all()
        assert err <= tol
