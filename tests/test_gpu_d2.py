"""The one-task D = 2 search (64 x 64 tiles of G, 16 rows a wave) against the
oracle's exhaustive top-k: edges of tiles and row blocks, constant and
dependent columns, noise and exact targets, rank ranges, search grids, and the
precision forms' matrices."""
import math

import numpy as np
import pytest

import oracle
from tests.parity import compare_topk
from tests.test_gpu_bound import problem, search

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["planted", "noise", "dependent", "constant", "exact"])
@pytest.mark.parametrize("S", [2, 3, 15, 16, 17, 63, 64, 65, 129, 200, 321])
def test_d2(kind, S):
    p = problem(kind, S, 1, 2, 8000 + S)
    k = max(1, min(20, math.comb(S, 2) // 2))
    print(f"{kind} S={S}", flush=True)
    gi, gs, _ = search(p, 2, k)
    oi, os_, _ = oracle.topk(p.F, p.y, 2, k, p.task_offsets)
    compare_topk(p, 2, k, gi, gs, oi, os_)


@pytest.mark.parametrize("kind", ["planted", "noise"])
def test_d2_grids_and_ranges(kind):
    S, k = 330, 15
    p = problem(kind, S, 1, 2, 8900)
    ref = search(p, 2, k)
    for grid in (1, 3, 8, 2048):
        for a, b in zip(ref, search(p, 2, k, grid=grid)):
            assert np.array_equal(a, b), grid
    for lo, hi in ((0, 1), (100, 140), (S - 8, S - 1)):
        r0 = sum(S - 1 - i for i in range(lo))
        r1 = sum(S - 1 - i for i in range(hi))
        kk = min(k, r1 - r0)
        gi, gs, _ = search(p, 2, kk, rng=(r0, r1))
        oi, os_, _ = oracle.topk(p.F, p.y, 2, kk, p.task_offsets, i1_range=(lo, hi))
        compare_topk(p, 2, kk, gi, gs, oi, os_)


@pytest.mark.parametrize("form", ["bf16", "fp16", "fp32"])
@pytest.mark.parametrize("kind", ["planted", "noise"])
@pytest.mark.parametrize("S", [65, 200])
def test_d2_precision_forms(S, kind, form):
    """The sliced Grams' matrices, and the FP32 solve.  Their errors (1e-6 of a
    correlation and of c) are far below the margin of the extra candidates that
    are re-scored in FP64, so the list is the oracle's to the FP64 tolerance."""
    from paper_2502_20072_amd import L0Search, _binding as B
    prec = {"bf16": B.SISSO_PREC_BF16_COMP, "fp16": B.SISSO_PREC_FP16_COMP, "fp32": B.SISSO_PREC_FP32_SOLVE}[form]
    p = problem(kind, S, 1, 2, 8500 + S)
    k = 20
    print(f"{form} {kind} S={S}", flush=True)
    s = L0Search(p.F, p.y, p.task_offsets, D_max=2, k_max=k, precision=prec)
    s.gram()
    s.search(2, k)
    gi, gs, _ = s.topk()
    s.close()
    oi, os_, _ = oracle.topk(p.F, p.y, 2, k, p.task_offsets)
    compare_topk(p, 2, k, gi, gs, oi, os_)
