"""What the other files check at sizes of one product kernel, in the others:
32 x 32 tiles (M <= 896; FP64 1280), 64 x 64 tiles, and, for 16-bit encodings
above M = 3008, pairs of 128 x 128 tiles.

  * one update against the oracle within the bounds of the kernel's own
    accumulation (path_bounds): every encoding in every kernel, HPCP and PMCP;
  * the accuracy that the FP64 totals and the fold of the 64 x 64 tiles are
    there for;
  * the guesses and the hole recursion in the 64 x 64 tiles;
  * schedules from tiles to tiles and from pairs to tiles;
  * recomputed segments and the loop's options, bitwise.
"""
import numpy as np
import pytest

import bounds
import oracle
import workloads
from path_bounds import path_kappa

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_1512_07236_amd as gcp  # noqa: E402
from test_gpu_elementwise import ENCODINGS, _oracle, check_step, gpu_iterates, log  # noqa: E402,F401


@pytest.fixture(scope="module")
def spectral():
    made = {}

    def make(M, N, seed=0):
        key = (M, N, seed)
        if key not in made:
            made[key] = workloads.spectral(M, N, gap=0.1, seed=M + seed)
        return made[key]
    return make


def solve(w, **opts):
    log(f"[gpu] {w.name} {opts}")
    with gcp.Context(w.M, **opts) as ctx:
        ctx.init(torch.from_numpy(w.H).cuda(), w.N, w.emin, w.emax)
        D, r = ctx.purify()
        return D.cpu().numpy(), r


def error(D, ref):
    return float(np.linalg.norm(D - ref) / np.sqrt(len(D)))


# ------------------------------------------------------------ one update
KERNELS = [(M, N, p) for M, N in ((20, 8), (385, 150)) for p in ENCODINGS]
KERNELS += [(1473, 560, p) for p in ENCODINGS]
KERNELS += [(3050, 1200, p) for p in ("bf16", "fp16", "bf16x3", "fp16x3", "bf16x6")]


@pytest.mark.parametrize("M,N,precision", KERNELS)
def test_one_update_within_the_kernels_own_bounds(M, N, precision, spectral, monkeypatch):
    monkeypatch.setattr(bounds, "accumulation_kappa", path_kappa)
    w = spectral(M, N, 5)
    log(f"[gpu] {precision} M={M}")
    it, hist = gpu_iterates(w, precision, [0])
    check_step(it[0], it[1], hist[0], precision, label=f"{precision} M={M}")


@pytest.mark.parametrize("M,N,precision", [(1473, 900, "fp64"), (1473, 900, "fp16x3"),
                                           (3050, 1900, "fp16x3")])
def test_one_pmcp_update_within_the_kernels_own_bounds(M, N, precision, spectral, monkeypatch):
    """Both branches of the coefficients: c_0 > 1/2 here, and c <= 1/2 from the
    hole side (the same spectrum reflected)."""
    monkeypatch.setattr(bounds, "accumulation_kappa", path_kappa)
    seen = set()
    for n_occ in (N, M - N):
        w = spectral(M, n_occ, 6)
        log(f"[gpu] pmcp {precision} M={M} N={n_occ}")
        it, hist = gpu_iterates(w, precision, [0], method="pmcp")
        c = hist[0][4]
        seen.add(bool(c > 0.5))
        ref, _ = oracle.update_at(it[0], c, "pmcp")
        b = bounds.step_bounds(it[0], c, precision, method="pmcp")
        diff = np.abs(it[1] - ref)
        log(f"  c={c:.3f} worst ratio {(diff / b['dD']).max():.3f}")
        assert np.all(diff <= b["dD"])
    assert seen == {False, True}


# -------------------------------------------------------------- accuracy
@pytest.mark.parametrize("precision", ["fp16x3", "bf16x6"])
def test_folds_and_fp64_totals_of_the_64_tiles(precision, spectral):
    """M = 2500, roundings of a term (one per MFMA product of 32 K values and
    one per FP32 addition), FP16X3 / BF16X6: the tiles 3 x 2 + 4 = 10 / 16 (two
    stages to a chunk, four chunks to an FP64 addition); one accumulator over
    80 stages 240 / 480; pairs in two splits of 40 stages, folded every 4 / 3,
    12 + 10 = 22 / 18 + 14 = 32; the tiles with an FP32 total instead of the
    FP64 one 6 + 40 = 46 / 12 + 40 = 52.  So the tiles err less than the split
    pairs, and would err more without their FP64 totals.  Against one
    accumulator the ratio is sqrt(24) = 4.9 / sqrt(30) = 5.5 in the accumulated
    rounding; the encoding's share is the same, so at least 2 in all."""
    w = spectral(2500, 1000, 7)
    ref = oracle.projector_from_spectrum(w.Q, w.lam, w.N)
    e = {}
    for name, opts in (("tiles", {}), ("one accumulator", {"fold_every": 1000}),
                       ("split pairs", {"ksplit": 2})):
        D, r = solve(w, precision=precision, tol_ddbar=1e-5, **opts)
        assert r.status in gcp.SUCCESS
        e[name] = error(D, ref)
        log(f"  {precision} {name}: p={r.iters} err={e[name]:.3e}")
    assert e["tiles"] < e["split pairs"]
    assert e["tiles"] < e["one accumulator"] / 2


# ------------------------------------------------------ variants, 64 tiles
@pytest.mark.parametrize("opts,N", [({"init": "search"}, 60), ({"init": "search"}, 65),
                                    ({"init": "hp", "alpha": 0.5}, 650),
                                    ({"hole": True}, 900), ({"method": "pmcp"}, 500)])
def test_variants_in_the_64_tiles_match_the_oracle(opts, N, spectral):
    """The searched guess with N = 65 is a runaway: both break down, after the
    same update, at the same iterate."""
    M = 1300
    w = spectral(M, N, 8)
    ref = oracle.purify_ex(w.H, N, w.emin, w.emax, tol_ddbar=1e-8, **opts)
    D, r = solve(w, precision="fp64", tol_ddbar=1e-8, **opts)
    assert r.status == {oracle.OK: gcp.OK, oracle.BREAKDOWN: gcp.ERR_BREAKDOWN}[ref.status]
    assert (ref.status == oracle.BREAKDOWN) == (N == 65) and r.iters == ref.iters
    assert np.abs(D - ref.D).max() < 1e-11
    assert abs(r.t1 - N) < 1e-10


# -------------------------------------------------------------- schedules
@pytest.mark.parametrize("M,N", [(1473, 560), (3050, 1200)])
@pytest.mark.parametrize("late", ["bf16x6", ""])
def test_schedules_into_the_64_tiles(M, N, late, spectral):
    """FP16X3, in tiles or in pairs (the padding is then a multiple of 256 for
    both phases), into FP64 tiles, directly or by way of BF16X6: the trace is
    exact throughout, the result idempotent to FP64 level, its error the
    early phase's (1e-6 at these sizes)."""
    w = spectral(M, N, 9)
    ref = oracle.projector_from_spectrum(w.Q, w.lam, w.N)
    opts = {"late_precision": "fp64", "switch_ddbar": 1e-2}
    if late:
        opts = {"late_precision": late, "switch_ddbar": 1e-1, "final_precision": "fp64",
                "final_ddbar": 1e-2}
    D, r = solve(w, precision="fp16x3", tol_ddbar=1e-10, max_iter=60, **opts)
    err, idem = error(D, ref), float(np.linalg.norm(D @ D - D))
    log(f"  p={r.iters} launches {r.gemm_launches} err={err:.2e} idem={idem:.1e}")
    assert r.status == gcp.OK
    assert np.abs(r.col("t1") - N).max() < 1e-10
    assert err < 1e-6 and idem < 1e-9
    again, r2 = solve(w, precision="fp16x3", tol_ddbar=1e-10, max_iter=60, **opts)
    assert np.array_equal(again, D) and np.array_equal(r2.history, r.history, equal_nan=True)


# --------------------------------------------------------- bitwise equals
@pytest.mark.parametrize("opts,bwd", [
    ({"precision": "fp16x3", "tol_ddbar": 1e-6}, "fp32"),
    ({"precision": "fp64", "tol_ddbar": 1e-8}, "fp64"),
    ({"precision": "fp16x3", "late_precision": "fp64", "switch_ddbar": 1e-2, "tol_ddbar": 1e-9},
     "fp64")])
def test_recomputed_segments_in_the_64_tiles(opts, bwd, spectral):
    """M = 1473: 256 whole tiles and 44 split ones, in the forward, in the
    recomputed segments and in the adjoint."""
    w = spectral(1473, 560, 9)
    G = torch.from_numpy(workloads.sym_gaussian(w.M, 310)).cuda().to(
        torch.float64 if bwd == "fp64" else torch.float32)
    H = torch.from_numpy(w.H).cuda()
    got = []
    for ck in (0, 3):
        with gcp.Context(w.M, keep_iterates=True, bwd_precision=bwd, checkpoint_every=ck,
                         **opts) as ctx:
            ctx.init(H, w.N, w.emin, w.emax)
            D, r = ctx.purify()
            assert r.status in gcp.SUCCESS
            got.append((D, ctx.backward(G)[0]))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("M,N,precision", [(1473, 560, "fp64"), (1473, 560, "fp16x3"),
                                           (3050, 1200, "fp16x3")])
def test_loop_options_in_the_larger_kernels(M, N, precision, spectral):
    w = spectral(M, N, 9)
    opts = {"precision": precision, "tol_ddbar": 1e-5}
    D, r = solve(w, **opts)
    assert r.status == gcp.OK
    for more in ({"sync_every": 1}, {"sync_every": 9}, {"profile": True}, {"max_iter": 1001},
                 {"keep_iterates": True}):
        Dm, rm = solve(w, **opts, **more)
        assert np.array_equal(Dm, D) and rm.iters == r.iters
        assert np.array_equal(rm.history, r.history, equal_nan=True)
