"""The rounding counts of the product kernels (path_bounds): never above the
pair kernel's, which bounds.py takes at every size, and independent of K where
the 16-bit tiles go on in FP64."""
import pytest

from bounds import PLANES, accumulation_kappa
from path_bounds import path, path_kappa

SIZES = [1, 20, 64, 65, 385, 896, 897, 1280, 1281, 1473, 1750, 2500, 3008, 3009, 8192]


@pytest.mark.parametrize("precision", sorted(PLANES))
def test_counts_are_at_most_the_pair_kernels(precision):
    for M in SIZES:
        assert 0 < path_kappa(M, precision) <= accumulation_kappa(M, precision), M
    for fold in (1, 3, 1000):
        assert path_kappa(1473, precision, fold) <= accumulation_kappa(1473, precision, fold)


def test_paths_and_the_counts_of_the_fine_encodings():
    assert [path(M, "fp64") for M in (1280, 1281, 8192)] == ["t32", "t64", "t64"]
    assert [path(M, "fp16x3") for M in (896, 897, 3008, 3009)] == ["t32", "t64", "t64", "pair"]
    assert path(200, "bf16", ksplit=4) == "pair"
    # two stages of 3 (6) products of 32 K values, four FP32 additions, two roundings
    for M in (1473, 2500, 3008):
        assert path_kappa(M, "fp16x3") == 2 * 96 + 6
        assert path_kappa(M, "bf16x6") == 2 * 192 + 6
