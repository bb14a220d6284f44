"""host_syncs counts the waits of gcp_purify's loop with nothing enqueued
behind them, exactly: every update with sync_every = 1, one at the end of a
solve that runs ahead, every sync_every updates in gcp_purify_static, and the
checks of a precision schedule before its switch."""
import pytest

import paper_1512_07236_amd as gcp
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

# options, and the updates whose decisions end the solve beyond p: none when
# the traces of update p - 1 stop it, one when the square of D_p is needed
STOPS = [({"precision": "fp16x3", "tol_ddbar": 1e-5}, 0),
         ({"precision": "fp64", "tol_ddbar": 0.0, "tol_idem": 1e-10}, 1),
         ({"precision": "fp32", "max_iter": 7}, 1),
         ({"precision": "fp64", "max_iter": 0}, 1)]


def solve(**opts):
    w = workloads.spectral(200, 77, 0.1, 91)
    with gcp.Context(w.M, **opts) as ctx:
        ctx.init(torch.from_numpy(w.H).cuda(), w.N, w.emin, w.emax)
        return ctx.purify()[1]


@pytest.mark.parametrize("opts,square", STOPS)
def test_every_update_or_once_at_the_end(opts, square):
    r = solve(sync_every=1, **opts)
    assert r.host_syncs == r.iters + square
    for k in (2, 4, 50):
        assert solve(sync_every=k, **opts).host_syncs == 1


@pytest.mark.parametrize("opts,square", STOPS)
def test_static_solve_checks_every_sync_every_updates(opts, square):
    w = workloads.spectral(200, 77, 0.1, 91)
    H = torch.from_numpy(w.H).cuda()
    for k in (1, 3, 4, 50):
        _, _, r = gcp.purify_static(H, w.N, w.emin, w.emax, sync_every=k, **opts)
        assert r.host_syncs == -(-(r.iters + square) // k)


def test_schedule_checks_every_square_until_it_switches():
    opts = {"precision": "fp16x3", "late_precision": "fp64", "tol_ddbar": 1e-9}
    r = solve(sync_every=1, switch_ddbar=1e-2, **opts)
    t12 = abs(r.history[:, 1] - r.history[:, 2])
    s = int((t12 <= 1e-2).argmax())
    assert 0 < s < r.iters
    # the squares of updates 0 .. s and the one formed again after the switch
    squares = s + 2
    assert r.host_syncs == r.iters + squares
    for k in (2, 4):
        assert solve(sync_every=k, switch_ddbar=1e-2, **opts).host_syncs == squares + 1
    # a schedule that never switches: the square of every iterate, the last of
    # them void
    r = solve(switch_ddbar=0.0, **opts)
    assert r.host_syncs == r.iters + 1
