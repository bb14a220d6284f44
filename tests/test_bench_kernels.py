"""bench.py names the product kernel that the library runs at a size, in the
counter summary and in the roofline, and its source hash covers all of them."""
import json
import os
import re

import pytest

import bench
import paper_1512_07236_amd as gcp
from path_bounds import PLANES, path
from test_bench import COPY, STREAM, _write_counters, sandbox  # noqa: F401

SMALL = "void gcp::k_small<5, 4>(gcp::GemmArgs)"
TILE = "void gcp::k_tile<5>(gcp::GemmArgs)"
PAIR = "void gcp::k_gemm16<5>(gcp::GemmArgs)"


@pytest.mark.parametrize("precision", sorted(PLANES))
def test_the_kernel_is_chosen_by_size_as_in_the_library(precision):
    src = open(os.path.join(os.path.dirname(bench.__file__), "paper_1512_07236_amd", "csrc",
                            "gcp_api.hip")).read()
    body = src[src.index("static int product_path("):]
    pair = int(re.search(r"M > (\d+)\)\) return PATH_PAIR", body).group(1))
    fp64, other = map(int, re.search(r"GCP_FP64 \? (\d+) : (\d+)\) \? PATH_T32", body).groups())
    names = {"t32": "k_small", "t64": "k_tile", "pair": "k_gemm16"}
    for edge in (pair, fp64, other):
        for M in (edge, edge + 1):
            assert bench.product_kernel(gcp.Precision.parse(precision), M) == names[path(M, precision)]
    assert path(fp64, "fp64") == "t32" and path(fp64 + 1, "fp64") == "t64"
    assert path(other, "fp32") == "t32" and path(other + 1, "fp32") == "t64"
    assert path(pair, "bf16") == "t64" and path(pair + 1, "bf16") == "pair"


@pytest.mark.parametrize("scale,kernel,name", [(1, PAIR, "k_gemm16<5>"), (4, TILE, "k_tile<5>"),
                                               (16, SMALL, "k_small<5>")])
def test_counter_summary_takes_the_kernel_that_ran(sandbox, scale, kernel, name):  # noqa: F811
    copy_kib = bench.COPY_BYTES / 1024
    others = [(k, 9e6) for k in (SMALL, TILE, PAIR) if k != kernel]
    others.append((kernel.replace("<5", "<55"), 9e6))
    _write_counters(sandbox / "fetch", "FETCH_SIZE",
                    [(kernel, 3.0e4), (kernel, 0.0), (STREAM, copy_kib), *others])
    _write_counters(sandbox / "write", "WRITE_SIZE", [(kernel, 5.0e3), (COPY, copy_kib), *others])
    assert bench.summarize_pmc("fp16x3", scale, str(sandbox / "fetch"), str(sandbox / "write")) == 0
    d = json.load(open(sandbox / "profiles" / f"gemm_fp16x3_M{8192 // scale}_pmc.json"))
    assert d["kernel"] == name and d["FETCH_SIZE"]["launches"] == 1
    assert d["hbm_bytes_per_launch"] == pytest.approx(3.5e4 * 1024)


def test_source_hash_covers_every_product_kernel(tmp_path, monkeypatch):
    csrc = os.path.join("paper_1512_07236_amd", "csrc")
    os.makedirs(tmp_path / csrc)
    root = os.path.dirname(os.path.abspath(bench.__file__))
    for f in ("gcp_kernels.hip", "gcp_encode.h", "gcp_mma.h", "gcp_kernels.h", "gcp_posts.h"):
        (tmp_path / csrc / f).write_text(open(os.path.join(root, csrc, f)).read())
    want = bench.product_kernel_hash()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.product_kernel_hash() == want
    path_ = tmp_path / csrc / "gcp_kernels.hip"
    text = path_.read_text()
    for mark in ("finish_rows(", "void k_tile(", "void k_small(", "void k_gemm16("):
        assert mark in text
        path_.write_text(text.replace(mark, "/**/" + mark, 1))
        assert bench.product_kernel_hash() != want
