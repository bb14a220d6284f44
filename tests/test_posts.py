"""The numbers by which the host waits for a context's reductions (gcp_posts.h)
over their whole range, compiled for the CPU: solves start anew in between,
and the count passes 2^31 and wraps at 2^32.  A wait before the post must not
be over, one for a posted number or an older one must be."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1512_07236_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "gcp_posts.h"
using namespace gcp;

int main(int, char **v) {
  uint32_t seq = (uint32_t)std::strtoul(v[1], nullptr, 10);
  Scalars host{};
  host.seq = seq;   // as gcp_create leaves it
  for (int solve = 0; solve < 6; ++solve) {
    host = start_scalars(0.4 * solve, 0.3, seq);
    if (host.t1 != 0.4 * solve || host.t2 != 0.3 || host.status != 0 || host.iter != 0 ||
        host.on_traces != 0 || !(host.prev_ddbar > 1e300))
      return std::printf("solve %d starts wrong\n", solve), 1;
    // reductions enqueued up to four ahead of the one that posts next
    uint32_t enqueued = seq;
    for (int k = 0; k < 40; ++k) {
      while ((int32_t)(enqueued - (seq + k)) < 4) ++enqueued;
      const uint32_t next = seq + k + 1;
      for (uint32_t q = next; q != enqueued + 1; ++q)
        if (posted(host.seq, q))
          return std::printf("solve %d: %u taken as posted at %u\n", solve, q, host.seq), 1;
      host.seq = next;
      if (!posted(host.seq, next) || !posted(host.seq, next - 1))
        return std::printf("solve %d: %u not posted at %u\n", solve, next, host.seq), 1;
    }
    seq = enqueued;   // the last few are void and never post
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("posts")
    (d / "posts.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC,
                           str(d / "posts.cpp"), "-o", str(d / "posts")])
    return str(d / "posts")


@pytest.mark.parametrize("first", [0, 2 ** 31 - 100, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 1, 3 * 2 ** 30,
                                   2 ** 32 - 64, 2 ** 32 - 1])
def test_waits_over_the_whole_range_of_numbers(program, first):
    r = subprocess.run([program, str(first)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.gpu
@pytest.mark.parametrize("opts", [{}, {"precision": "fp16x3", "late_precision": "fp64",
                                       "switch_ddbar": 1e-2},
                                  {"keep_iterates": True, "checkpoint_every": 3},
                                  {"max_iter": 0}])
def test_a_context_solves_on_across_the_wrap(opts):
    """A context's numbers wrap within its first solves; every one of many
    solves, with gcp_init (and a checkpointed backward) in between, is bitwise
    the first."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np
    import paper_1512_07236_amd as gcp
    import workloads
    w = workloads.spectral(100, 38, 0.1, 93)
    H = torch.from_numpy(w.H).cuda()
    with gcp.Context(w.M, tol_ddbar=1e-9, **opts) as ctx:
        first = None
        for _ in range(40):
            ctx.init(H, w.N, w.emin, w.emax)
            D, r = ctx.purify()
            got = [D, ctx.backward(H)[0]] if opts.get("keep_iterates") else [D]
            if first is None:
                first, r0 = got, r
                assert r.status == (gcp.ERR_NOT_CONVERGED if "max_iter" in opts else gcp.OK)
            assert r.status == r0.status and r.iters == r0.iters
            assert np.array_equal(r.history, r0.history, equal_nan=True)
            assert all(torch.equal(a, b) for a, b in zip(got, first))
