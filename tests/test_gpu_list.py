"""Prefix-list search and score selection: the list's pooled bound (repeated,
malformed and rank-deficient rows, lists longer than the pool takes) against
the oracle's exhaustive top-k, and the selection's cut over the histogram's
edges against the sorted scores."""
import itertools
import math

import numpy as np
import pytest

import oracle
from synth.problems import tiny_problem
from tests.parity import compare_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("S,D,kind", [(40, 2, "plain"), (30, 3, "plain"), (96, 3, "plain"), (14, 4, "plain"),
                                      (30, 3, "repeated"), (14, 4, "repeated"), (30, 3, "dependent"),
                                      (14, 4, "dependent")])
def test_list_of_all_prefixes(S, D, kind, T):
    """Every (D-1)-prefix in the list (S = 96, D = 3: 4560 rows): the result
    is the exhaustive one, whatever repeats and invalid rows are among them."""
    import torch
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    p = tiny_problem(6100 + S + D + T, S=S, n=45 * T, T=T, D=D, sigma=0.3)
    if kind == "dependent":
        for j in range(3, S, 5):
            p.F[j] = 2.0 * p.F[j - 1]
        p.F[S - 2] = 0.5
    pre = np.array(list(itertools.combinations(range(S), D - 1)), dtype=np.int32)
    rng = np.random.default_rng(S)
    if kind == "repeated":
        bad = np.full((5, D - 1), S, dtype=np.int32)
        bad[1:3] = -1
        pre = np.concatenate([np.repeat(pre, 3, axis=0), bad])
    pre = pre[rng.permutation(len(pre))]
    k = min(25, math.comb(S, D) // 3)
    s = L0Search(p.F, p.y, p.task_offsets, D_max=D, k_max=k)
    s.gram()
    B.sisso_l0_search_list(s.handle, D, k, torch.from_numpy(pre).to("cuda"))
    s.last_D, s.last_k = D, k
    gi, gs, _ = s.topk()
    s.close()
    oi, os_, _ = oracle.topk(p.F, p.y, D, k, p.task_offsets)
    compare_topk(p, D, k, gi, gs, oi, os_)


@pytest.mark.parametrize("grid", [1, 3, 1024])
@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("S,D", [(40, 2), (20, 3), (14, 4)])
def test_copies_do_not_fill_a_list(S, D, T, grid):
    """A few rows repeated many times come first: a wave that reaches their
    tuples again and again still takes the better ones of the rows behind."""
    import torch
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    p = tiny_problem(6300 + S + T, S=S, n=45 * T, T=T, D=D, sigma=0.3)
    pre = np.array(list(itertools.combinations(range(S), D - 1)), dtype=np.int32)
    head = pre[np.random.default_rng(S).permutation(len(pre))[:4]]
    pre = np.concatenate([np.tile(head, (50, 1)), pre])
    k = 48
    s = L0Search(p.F, p.y, p.task_offsets, D_max=D, k_max=k)
    s.set_search_grid(grid)
    s.gram()
    B.sisso_l0_search_list(s.handle, D, k, torch.from_numpy(pre).to("cuda"))
    s.last_D, s.last_k = D, k
    gi, gs, _ = s.topk()
    s.close()
    oi, os_, _ = oracle.topk(p.F, p.y, D, k, p.task_offsets)
    compare_topk(p, D, k, gi, gs, oi, os_)


@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("S,reps", [(64, 1), (65, 1), (66, 1), (33, 2), (34, 2), (129, 2), (130, 2), (130, 5)])
def test_merge_of_copies(S, reps, T):
    """Four rows (one feature each), each up to five times: 252 to 2580
    candidates reach the merge, the six pairs of the four features from two
    rows, all of them `reps` times.  Either side of what is ranked by counting
    (256 candidates) and of the sort's batches (1024)."""
    import torch
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    p = tiny_problem(6400 + S + T, S=S, n=45 * T, T=T, D=2, sigma=0.3)
    pre = np.tile(np.arange(4, dtype=np.int32)[:, None], (reps, 1))
    k = min(480, 4 * (S - 1) - 6)
    s = L0Search(p.F, p.y, p.task_offsets, D_max=2, k_max=k)
    s.gram()
    B.sisso_l0_search_list(s.handle, 2, k, torch.from_numpy(pre).to("cuda"))
    s.last_D, s.last_k = 2, k
    gi, gs, _ = s.topk()
    s.close()
    oi, os_, _ = oracle.topk(p.F, p.y, 2, k, p.task_offsets, i1_range=(0, 4))
    compare_topk(p, 2, k, gi, gs, oi, os_)


@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("D", [2, 3, 4])
def test_empty_list(D, T):
    """A list without rows has no tuples: every result row is marked empty."""
    import torch
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    p = tiny_problem(6200 + D, S=20, n=45 * T, T=T, D=D, sigma=0.3)
    s = L0Search(p.F, p.y, p.task_offsets, D_max=D, k_max=5)
    s.gram()
    B.sisso_l0_search_list(s.handle, D, 5, torch.empty((0, D - 1), dtype=torch.int32, device="cuda"))
    s.last_D, s.last_k = D, 5
    gi, gs, gc = s.topk()
    assert s.scored() == 0
    s.close()
    assert (gi == -1).all() and np.isposinf(gs).all() and np.isnan(gc).all()


@pytest.mark.parametrize("n,K", [(1, 1), (5, 3), (1024, 1024), (5000, 1), (5000, 4999), (100003, 700)])
@pytest.mark.parametrize("kind", ["normal", "equal", "negative", "nan", "infinite"])
def test_selection_cut(n, K, kind):
    """The K largest scores are all selected, and nothing below the K-th by
    more than 2^8 steps of the key."""
    import torch
    from paper_2502_20072_amd import _binding as B
    rng = np.random.default_rng(n + K)
    sc = rng.standard_normal(n).astype(np.float32)
    if kind == "equal":
        sc[:] = 0.25
    elif kind == "negative":
        sc = -np.abs(sc) - 1e-3
    elif kind == "nan":
        sc[rng.random(n) < 0.3] = np.nan
    elif kind == "infinite":
        sc[rng.random(n) < 0.2] = -np.inf
        sc[rng.random(n) < 0.1] = np.inf
    t = torch.from_numpy(sc).to("cuda")
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    ws = torch.empty(B.sisso_select_workspace_bytes(), dtype=torch.uint8, device="cuda")
    cnt = B.sisso_select_top(t, K, out, ws, torch.cuda.current_stream().cuda_stream)
    got = np.sort(out[:cnt].cpu().numpy())
    u = sc.view(np.uint32).astype(np.int64)
    key = np.where(u & 0x80000000, 0xFFFFFFFF - u, u | 0x80000000)
    key[np.isnan(sc)] = -1
    order = np.sort(key[key >= 0])[::-1]
    if len(order) < K:                 # fewer numbers than K: all of them
        want = np.flatnonzero(key >= 0)
        assert np.array_equal(got, want)
        return
    kth = order[K - 1]
    assert len(np.unique(got)) == cnt >= K
    assert set(np.flatnonzero(key >= kth)) <= set(got.tolist())
    assert key[got].min() >= kth - 256
