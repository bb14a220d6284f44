"""The adjoint of a solve that a precision schedule's check stops before its
first update: D_0 is kept for the derivative of the guess, each time, and not
the one of an earlier solve in the same context."""
import numpy as np
import pytest

from oracle import grad
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1512_07236_amd as gcp  # noqa: E402
from test_gpu_adjoint import _oracle, rel_max, to_gpu  # noqa: E402,F401

SCHEDULE = {"precision": "fp64", "late_precision": "fp32", "switch_ddbar": 0.0}


@pytest.mark.parametrize("more", [{}, {"checkpoint_every": 2}])
def test_limit_of_no_update(more):
    """Two problems in one context, on either side of half filling (the second
    reads <Gbar_0, D_0>)."""
    with gcp.Context(200, keep_iterates=True, max_iter=0, **SCHEDULE, **more) as ctx:
        for N, seed in ((60, 25), (140, 26)):
            w = workloads.spectral(200, N, 0.1, seed)
            Gp = workloads.sym_gaussian(200, seed + 200)
            ctx.init(to_gpu(w.H), N, w.emin, w.emax)
            _, res = ctx.purify()
            assert res.iters == 0 and res.status == gcp.ERR_NOT_CONVERGED
            dH, _ = ctx.backward(to_gpu(Gp))
            ref = grad.adjoint(w.H, N, w.emin, w.emax, 0, Gp)
            assert rel_max(dH.cpu().numpy(), ref) <= 1e-13


@pytest.mark.parametrize("N", [0, 128])
def test_degenerate_filling(N):
    w = workloads.spectral(128, 64, 0.1, 27)
    with gcp.Context(128, keep_iterates=True, **SCHEDULE) as ctx:
        ctx.init(to_gpu(w.H), N, w.emin, w.emax)
        _, res = ctx.purify()
        assert res.iters == 0 and res.status == gcp.OK
        dH, _ = ctx.backward(to_gpu(workloads.sym_gaussian(128, 227)))
        assert np.all(dH.cpu().numpy() == 0.0)
