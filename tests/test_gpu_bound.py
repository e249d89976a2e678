"""The record-table searches' superset bound: a group of four first indices is
tested together (the fit on the group, j and k bounds its tuples' fits), and
only what passes is scored tuple by tuple.  Against the oracle's exhaustive
top-k over the edges of units (64 rows, 64 columns) and groups of 4, one
and several tasks, rank ranges, every pool distribution (search grids), and
inputs on which the bound is weak or cannot be used: noise targets, groups
with dependent or constant columns, columns in the span of others."""
import math

import numpy as np
import pytest

import oracle
from synth.problems import tiny_problem
from tests.parity import compare_topk

pytestmark = pytest.mark.gpu


def problem(kind, S, T, D, seed):
    p = tiny_problem(seed, S=S, n=40 * T + 7, T=T, D=D, sigma=30.0 if kind == "noise" else 0.2)
    rng = np.random.default_rng(seed)
    if kind == "dependent":
        for j in range(1, S, 5):
            p.F[j] = p.F[j - 1] + 1e-3 * p.F[j]        # close pairs inside a group
        for j in range(7, S, 9):
            p.F[j] = p.F[j - 3] - 2.0 * p.F[j - 6]     # columns in the span of two others
    elif kind == "constant":
        for j in range(2, S, 6):
            p.F[j, p.task_offsets[-2]:] = 1.5          # constant on the last task
        if S > 12:
            p.F[8:12] = 0.25                           # a whole group
    elif kind == "exact":
        idx = sorted(rng.choice(S, size=D, replace=False))
        p.y[:] = p.F[idx].sum(0)
    return p


def search(p, D, k, grid=None, rng=None):
    from paper_2502_20072_amd import L0Search
    s = L0Search(p.F, p.y, p.task_offsets, D_max=D, k_max=k)
    if grid:
        s.set_search_grid(grid)
    s.gram()
    (s.search_range(D, k, *rng) if rng else s.search(D, k))
    out = s.topk()
    s.close()
    return out


@pytest.mark.parametrize("kind", ["planted", "noise", "dependent", "constant", "exact"])
@pytest.mark.parametrize("S,T", [(5, 1), (9, 2), (64, 1), (66, 3), (67, 1), (129, 2), (131, 1), (195, 1)])
def test_d3(kind, S, T):
    p = problem(kind, S, T, 3, 3000 + S + T)
    k = min(20, math.comb(S, 3) // 2)
    print(f"{kind} S={S} T={T}", flush=True)
    gi, gs, gc = search(p, 3, k)
    oi, os_, _ = oracle.topk(p.F, p.y, 3, k, p.task_offsets)
    compare_topk(p, 3, k, gi, gs, oi, os_)


@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("kind", ["planted", "noise"])
def test_d3_grids_and_ranges(kind, T):
    """Every search grid gives the same result bit for bit, and a range of
    ranks the oracle's list of that range."""
    S, k = 140, 15
    p = problem(kind, S, T, 3, 77 + T)
    ref = search(p, 3, k)
    for grid in (1, 3, 8, 64, 2048):
        got = search(p, 3, k, grid=grid)
        for a, b in zip(ref, got):
            assert np.array_equal(a, b), grid
    # first indices [2, 5): a contiguous range of lexicographic ranks
    r0 = sum(math.comb(S - 1 - i, 2) for i in range(2))
    r1 = sum(math.comb(S - 1 - i, 2) for i in range(5))
    gi, gs, _ = search(p, 3, k, rng=(r0, r1))
    oi, os_, _ = oracle.topk(p.F, p.y, 3, k, p.task_offsets, i1_range=(2, 5))
    compare_topk(p, 3, k, gi, gs, oi, os_)


@pytest.mark.parametrize("T", [1, 2])
def test_search_in_several_passes(T):
    """S = 7200 takes two passes over the units (one holds 2^21).  Two of three
    columns are constant, so the result is that of the 2400 live columns
    alone, which take one pass."""
    p = tiny_problem(41 + T, S=2400, n=64 * T, T=T, D=3, k=30, sigma=0.3)
    ref = search(p, 3, 30)
    wide = tiny_problem(41 + T, S=3, n=64 * T, T=T, D=3, k=30)
    wide.F = np.full((7200, p.n), 0.5)
    wide.F[::3] = p.F
    wide.y, wide.task_offsets = p.y, p.task_offsets
    got = search(wide, 3, 30)
    assert np.array_equal(got[0], 3 * ref[0])
    assert np.array_equal(got[1], ref[1]) and np.array_equal(got[2], ref[2])


@pytest.mark.parametrize("kind", ["planted", "noise", "dependent", "constant", "exact"])
@pytest.mark.parametrize("S", [4, 5, 8, 9, 13, 65, 68, 71])
def test_d4(kind, S):
    """D = 4, one task: pairs of groups (the ten-feature fit bounds sixteen
    tuples), over the edges of groups, pairs and tiles."""
    p = problem(kind, S, 1, 4, 4000 + S)
    k = max(1, min(20, math.comb(S, 4) // 2))
    print(f"{kind} S={S}", flush=True)
    gi, gs, gc = search(p, 4, k)
    oi, os_, _ = oracle.topk(p.F, p.y, 4, k, p.task_offsets)
    compare_topk(p, 4, k, gi, gs, oi, os_)


@pytest.mark.parametrize("kind", ["planted", "noise", "dependent"])
def test_d4_grids_and_ranges(kind):
    """Every search grid gives the same result bit for bit; a range of ranks
    gives the oracle's list of that range, also one with fewer tuples than the
    list holds (no threshold: every unit is scored whole)."""
    S, k = 68, 15
    p = problem(kind, S, 1, 4, 91)
    ref = search(p, 4, k)
    for grid in (1, 3, 8, 64, 2048):
        got = search(p, 4, k, grid=grid)
        for a, b in zip(ref, got):
            assert np.array_equal(a, b), grid
    r0 = sum(math.comb(S - 1 - i, 3) for i in range(3))
    r1 = sum(math.comb(S - 1 - i, 3) for i in range(6))
    gi, gs, _ = search(p, 4, k, rng=(r0, r1))
    oi, os_, _ = oracle.topk(p.F, p.y, 4, k, p.task_offsets, i1_range=(3, 6))
    compare_topk(p, 4, k, gi, gs, oi, os_)
    # first index S - 6: C(5, 3) = 10 tuples
    r0 = sum(math.comb(S - 1 - i, 3) for i in range(S - 6))
    gi, gs, _ = search(p, 4, 10, rng=(r0, r0 + 10))
    oi, os_, _ = oracle.topk(p.F, p.y, 4, 10, p.task_offsets, i1_range=(S - 6, S - 5))
    compare_topk(p, 4, 10, gi, gs, oi, os_)


def test_d4_search_in_several_passes():
    """S = 760 takes two passes over the units (one holds 2^18).  Three of four
    columns are constant, so the result is that of the 190 live columns alone."""
    p = tiny_problem(45, S=190, n=80, D=4, k=30, sigma=0.3)
    ref = search(p, 4, 30)
    wide = tiny_problem(45, S=4, n=80, D=4, k=1)
    wide.F = np.full((760, p.n), 0.5)
    wide.F[::4] = p.F
    wide.y, wide.task_offsets = p.y, p.task_offsets
    got = search(wide, 4, 30)
    assert np.array_equal(got[0], 4 * ref[0])
    assert np.array_equal(got[1], ref[1]) and np.array_equal(got[2], ref[2])


def test_batch_of_weakly_bounded_problems():
    """The batched search takes the bound's flagged tuples inline: equal to
    the single searches bit for bit on planted, noise and dependent columns."""
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    ps = [problem(kind, S, 1, 3, 500 + S) for kind in ("planted", "noise", "dependent") for S in (33, 140)]
    hs = [L0Search(p.F, p.y, p.task_offsets, D_max=3, k_max=12) for p in ps]
    b = B.sisso_l0_batch_create([h.handle for h in hs], 3, 12)
    for _ in range(2):
        B.sisso_l0_batch_launch(b)
        for p, h in zip(ps, hs):
            h.last_D, h.last_k = 3, 12
            got, ref = h.topk(), search(p, 3, 12)
            for x, y in zip(got, ref):
                assert np.array_equal(x, y)
    B.sisso_l0_batch_destroy(b)
    for h in hs:
        h.close()
