"""The tile products at the sizes where their launch shape changes, one update
at a time against the oracle within the derived bounds: 32 x 32 tiles (every
encoding) with one row of them half empty, with fewer K stages than waves, and
with an odd row of padding; around the sizes at which 64 x 64 tiles take over,
where every tile is split along K; 300 of those, of which 44 are split; 406,
of which 150 are split over three blocks each; and
the two sides of the size at which the 16-bit encodings change to tile
pairs."""
import pytest

import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from test_gpu_elementwise import ENCODINGS, _oracle, check_guess, check_step, gpu_iterates, log  # noqa: E402,F401

CASES = [(M, N, p) for M, N in ((20, 8), (64, 24), (65, 30), (385, 150)) for p in ENCODINGS]
CASES += [(M, 350, p) for M in (896, 897) for p in ("fp32", "bf16", "fp16x3", "bf16x6")]
CASES += [(M, 500, "fp64") for M in (1280, 1281)]
CASES += [(1473, 560, p) for p in ("fp64", "fp32", "fp16x3", "bf16x6")]
CASES += [(1750, 700, p) for p in ("fp64", "fp32")]
CASES += [(M, 1200, p) for M in (3008, 3009) for p in ("fp16x3", "bf16x6")]


@pytest.mark.parametrize("M,N,precision", CASES)
def test_one_update_at_a_time_at_the_edges(M, N, precision):
    w = workloads.spectral(M, N, gap=0.1, seed=M + 3)
    log(f"[gpu] tiles {precision} M={M}")
    steps = [0, 1] if M < 3000 else [0]
    it, hist = gpu_iterates(w, precision, steps)
    check_guess(w, it[0], precision)
    for n in steps:
        check_step(it[n], it[n + 1], hist[n], precision, label=f"{precision} M={M}")
