"""The host side of a solve: decisions posted to pinned memory, the history
staged there when it is short, update 0 reading D_0 in place, kept iterates
allocated several at a time.  None of it may change a result: every variant
is bitwise the plain solve, whatever ran before in the same context."""
import threading

import numpy as np
import pytest

import oracle
import paper_1512_07236_amd as gcp
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)


def context(w, **opts):
    ctx = gcp.Context(w.M, **opts)
    ctx.init(torch.from_numpy(w.H).cuda(), w.N, w.emin, w.emax)
    return ctx


def same(a, b):
    return (torch.equal(a[0], b[0]) and a[1].status == b[1].status and a[1].iters == b[1].iters
            and np.array_equal(a[1].history, b[1].history, equal_nan=True))


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-9), ("fp16x3", 1e-5)])
@pytest.mark.parametrize("opts", [
    {"max_iter": 1000},            # the longest history staged in pinned memory
    {"max_iter": 1001},            # the shortest that is not
    {"sync_every": 1}, {"sync_every": 2}, {"sync_every": 9},
    {"keep_iterates": True},       # D_0 copied, one iterate kept per update
    {"keep_iterates": True, "checkpoint_every": 3},
    {"profile": True},
])
def test_variants_are_bitwise_the_plain_solve(precision, tol, opts):
    w = workloads.spectral(200, 77, 0.1, 91)
    with context(w, precision=precision, tol_ddbar=tol) as ctx:
        plain = ctx.purify()
        assert plain[1].status == gcp.OK
        assert same(ctx.purify(), plain)       # D_0 is still there
    with context(w, precision=precision, tol_ddbar=tol, **opts) as ctx:
        for _ in range(2):
            assert same(ctx.purify(), plain)
        ctx.init(torch.from_numpy(w.H).cuda(), w.N, w.emin, w.emax)
        assert same(ctx.purify(), plain)


@pytest.mark.parametrize("opts", [{}, {"keep_iterates": True}])
def test_stops_at_the_guess_and_at_the_limit(opts):
    """max_iter = 0 returns D_0 (no update reads or writes it); a limit below
    the convergence returns that iterate; both leave D_0 in place."""
    w = workloads.spectral(200, 77, 0.1, 91)
    got = []
    for _ in range(2):
        for n in (0, 1, 3):
            with context(w, max_iter=n, **opts) as ctx:
                D, r = ctx.purify()
                assert r.iters == n and r.status == gcp.ERR_NOT_CONVERGED
                assert same(ctx.purify(), (D, r))
                got.append(D.cpu().numpy())
    for a, b in zip(got[:3], got[3:]):
        assert np.array_equal(a, b)
    # one update of the oracle's recursion leads from each to the next
    step, _ = oracle.update_at(got[0], float(r.history[0][4]))
    # rows of norm at most one: each sum of 200 products errs by at most 200 u,
    # weighted 2 + 2c <= 4 and 2 (twice, X2 and X2 D), on both sides
    assert np.abs(step - got[1]).max() <= 2 * 8 * 210 * 2.0 ** -53


def test_two_contexts_on_two_threads_and_streams():
    """Each context polls its own posts: solves side by side are bitwise the
    solves one after the other."""
    works = [workloads.spectral(200, 77, 0.1, 91), workloads.spectral(333, 120, 0.1, 92)]
    alone = []
    for w in works:
        with context(w, precision="fp16x3", tol_ddbar=1e-5) as ctx:
            alone.append(ctx.purify())
    torch.cuda.synchronize()
    ok = [0, 0]

    def body(k):
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for _ in range(10):
                with context(works[k], precision="fp16x3", tol_ddbar=1e-5) as ctx:
                    got = ctx.purify()
                stream.synchronize()
                ok[k] += same(got, alone[k])

    threads = [threading.Thread(target=body, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert ok == [10, 10]
