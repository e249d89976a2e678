"""The threshold pre-pass: its bound theta0 is an upper bound of the KP-th
best SSE (KP = 64 candidates are kept for k = 10), is at most one histogram
bin above the KP-th best of the tuples it has scored, and the search that
starts from it returns the tuples of a plain FP64 evaluation of every tuple.
Sizes: fewer tuples than KP, workgroup edges of the extension (256 features
per workgroup), more features than the selection sorts (4096), one and
several tasks."""
import itertools

import numpy as np
import pytest

from synth.problems import tiny_problem

pytestmark = pytest.mark.gpu


def all_sse(p, tuples):
    """SSE of every tuple summed over tasks (normal equations of the centred
    columns in FP64; well-conditioned Gaussian columns)."""
    tot = np.zeros(len(tuples))
    for a, b in zip(p.task_offsets[:-1], p.task_offsets[1:]):
        x = p.F[:, a:b] - p.F[:, a:b].mean(1, keepdims=True)
        yc = p.y[a:b] - p.y[a:b].mean()
        G, v = x @ x.T, x @ yc
        A, r = G[tuples[:, :, None], tuples[:, None, :]], v[tuples]
        tot += yc @ yc - (np.linalg.solve(A, r[:, :, None])[:, :, 0] * r).sum(1)
    return tot


@pytest.mark.parametrize("S,D,T", [(5, 2, 1), (12, 2, 1), (255, 2, 1), (257, 2, 2), (513, 2, 1), (4200, 2, 1),
                                   (9, 3, 1), (64, 3, 1), (65, 3, 3), (13, 4, 1), (33, 4, 1), (24, 4, 2)])
def test_bound_and_search(S, D, T):
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    p = tiny_problem(seed=900 + S + 7 * D + T, S=S, n=40 * T + S % 7, T=T, D=D, k=10, sigma=0.5)
    if D == 2:
        tuples = np.stack(np.triu_indices(S, 1), 1)
    else:
        tuples = np.array(list(itertools.combinations(range(S), D)))
    sse = all_sse(p, tuples)
    order = np.argsort(sse, kind="stable")
    k = min(10, len(tuples))
    s = L0Search(p.F, p.y, p.task_offsets, D_max=D, k_max=k)
    idx, got, _ = s.gram().search(D, k).topk()
    theta0 = B.sisso_l0_search_stats(s.handle)["theta0"]
    KP = 64
    if len(tuples) < KP:
        assert theta0 == np.inf
    else:
        # SSEs of Gaussian columns from normal equations: relative error far below 1e-9
        assert theta0 >= sse[order[KP - 1]] * (1 - 1e-9)
        # the pool holds at least one prefix's S - D + 1 tuples, so with KP
        # of them theta0 is finite
        if S - D + 1 >= KP:
            assert theta0 < np.inf
    assert np.array_equal(idx, tuples[order[:k]])
    np.testing.assert_allclose(got, sse[order[:k]], rtol=1e-9)


def test_bound_is_near_the_kth_best_of_a_planted_pair():
    """Pairs of a planted problem: every one of the 64 best pairs holds one of
    the eight most relevant features, so the pool holds them all and theta0 is
    their 64th SSE rounded up by at most one bin (1/64)."""
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    p = tiny_problem(seed=77, S=300, n=200, D=2, k=10, planted=[17, 240], sigma=0.1)
    tuples = np.stack(np.triu_indices(300, 1), 1)
    sse = all_sse(p, tuples)
    rel = np.argsort(-np.abs((p.F - p.F.mean(1, keepdims=True)) @ (p.y - p.y.mean())) / p.F.std(1))[:8]
    order = np.argsort(sse)
    assert all(set(t) & set(rel) for t in tuples[order[:64]])  # the premise
    s = L0Search(p.F, p.y, D_max=2, k_max=10)
    s.gram().search(2, 10).topk()
    theta0 = B.sisso_l0_search_stats(s.handle)["theta0"]
    kth = sse[order[63]]
    assert kth * (1 - 1e-9) <= theta0 <= kth * (1 + 1 / 64 + 1e-9)
