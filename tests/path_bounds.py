"""Rounding steps of a product term in each of the product kernels (test
helper; the bounds themselves are those of ``bounds``, whose own count is that
of the pair kernel at every size and so an upper bound for the others).

  * 32 x 32 tiles: four waves take every fourth K stage each; a wave folds its
    chunk accumulator into its FP32 total, and the four totals are added in
    FP64.
  * 64 x 64 tiles: FP64 and FP32 split the K values of a stage over two wave
    groups, whose totals are added once; the 16-bit encodings move their FP32
    totals on into FP64 ones every four folds.  A tile split along K adds its
    partial tiles in FP64, each rounded once when it is published.
  * pairs of 128 x 128 tiles: as ``bounds.accumulation_kappa``.

FP64 additions behind FP32 totals are below first order here.
"""
from __future__ import annotations

import math

from bounds import PLANES, PRODUCTS, accumulation_kappa

GF = 4   # folds between two FP64 additions in the 16-bit 64 x 64 tiles


def path(M: int, precision: str, ksplit: int = 0) -> str:
    """Product kernel at size M: "t32", "t64" or "pair"."""
    if precision not in ("fp64", "fp32") and (ksplit >= 2 or M > 3008):
        return "pair"
    return "t32" if M <= (1280 if precision == "fp64" else 896) else "t64"


def _half_up(x: float) -> int:
    return max(1, math.floor(x + 0.5))


def path_kappa(M: int, precision: str, fold_every: int = 0, ksplit: int = 0) -> int:
    p = path(M, precision, ksplit)
    if p == "pair":
        return accumulation_kappa(M, precision, fold_every, ksplit)
    Mp = (M + 63) // 64 * 64
    if precision == "fp64":
        # a quarter of K and the four sums; half of K, the halves, 16 splits
        return Mp // 4 + 4 if p == "t32" else Mp // 2 + 1 + 16
    planes = PLANES[precision]
    if precision == "fp32":
        stages, per_stage, terms = Mp // 32, 8, 32   # 32 K values in steps of four
    else:
        stages = Mp * planes // 64 if planes <= 2 else Mp // 32
        per_stage = 2 if planes == 1 else PRODUCTS[precision]
        terms = 32 * per_stage
    if p == "t32":
        fold = fold_every or _half_up(math.sqrt(stages / 4 / per_stage))
        if not fold_every and precision in ("bf16", "fp16", "bf16x3"):
            fold = max(fold, 2)
        own = -(-stages // 4)
        fold = min(fold, own)
        return terms * fold + math.ceil(own / fold) + 1
    worst = 0
    for splits in range(1, 17):   # a product whose tiles are all split folds one split's stages
        own = -(-stages // splits)
        fold = fold_every or _half_up(math.sqrt(own / per_stage))
        if not fold_every and precision in ("fp16x3", "bf16x6"):
            fold = min(fold, 2)
        fold = min(fold, own)
        if precision == "fp32":   # a wave's half of every stage; the halves, the partial
            kappa = terms // 2 * fold + math.ceil(own / fold) + 2
        else:
            kappa = terms * fold + min(GF, math.ceil(own / fold)) + 2
        worst = max(worst, kappa)
    return worst
