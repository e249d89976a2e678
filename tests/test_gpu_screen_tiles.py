"""Screening over the edges of its tiles (16 samples, two a lane; residuals
taken from registers) and the exact selection's early end, against
oracle/sisso_ref.py: task lengths around one and two tiles, odd row lengths
(columns at odd multiples of 8 bytes), groups with one and with several first
children, every padded residual count, values that are not finite in the
first, a middle and the last sample."""
import itertools

import numpy as np
import pytest

from oracle import sisso_ref as R

pytestmark = pytest.mark.gpu


def _d(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("op", ["stored", "add", "div", "sq"])
@pytest.mark.parametrize("lengths,nres", [((15,), 1), ((16,), 2), ((17,), 3), ((31,), 1), ((32,), 10), ((33,), 16),
                                          ((47,), 5), ((48, 5), 2), ((16, 33), 10), ((101, 64, 31), 8)])
def test_tile_edges(op, lengths, nres):
    import torch
    from paper_2502_20072_amd import _binding as B
    n, Mc = sum(lengths), 13
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    rng = np.random.default_rng(n + nres)
    X = rng.normal(size=(Mc, n)) + 2.0
    X[4, 0] = np.inf
    X[5, n // 2] = np.nan
    X[6, n - 1] = -np.inf
    res = np.array([X[r % 4] * 0.4 + rng.normal(size=n) for r in range(nres)])
    h = B.SisScreen(_d(res), off)
    if op == "stored":
        sc = torch.empty(Mc, dtype=torch.float64, device="cuda:0")
        h.score(_d(X), sc)
        ref = R.sis_scores(X, list(res), off)
        got = sc.cpu().numpy()
        ok = np.isfinite(ref)
    else:
        # the first 64 candidates share their first child, the rest do not
        pairs = [(0, 1 + i % (Mc - 1)) for i in range(64)] + list(itertools.combinations(range(Mc), 2))
        pairs = np.array(pairs, dtype=np.int32)
        lo, hi = 1e-5, 1e8
        vals, ok = R.create(op, X, pairs, lo, hi)
        sc = torch.empty(len(pairs), dtype=torch.float64, device="cuda:0")
        v = torch.empty(len(pairs), dtype=torch.uint8, device="cuda:0")
        h.score_op(op, _d(X), _d(pairs), lo, hi, sc, v)
        got = sc.cpu().numpy()
        assert v.cpu().numpy().astype(bool).tolist() == ok.tolist()
        ref = np.array([R.sis_score(vals[p], list(res), off) if ok[p] else np.nan for p in range(len(pairs))])
    h.close()
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    live = ~np.isnan(ref)
    np.testing.assert_allclose(got[live], ref[live], rtol=0, atol=1e-12)


@pytest.mark.parametrize("M,m", [(5, 5), (5, 1), (4097, 4096), (50000, 3), (50000, 50)])
@pytest.mark.parametrize("kind", ["distinct", "bits", "equal", "mixed"])
def test_selection_ends_early(M, m, kind):
    """Scores that are told apart by their first digit, by their last bits,
    or by their index only."""
    import torch
    from paper_2502_20072_amd import _binding as B
    rng = np.random.default_rng(M + m)
    if kind == "distinct":
        sc = np.ldexp(rng.uniform(1, 2, M), rng.integers(-400, 400, M))
    elif kind == "bits":
        sc = (np.float64(0.5).view(np.int64) + rng.permutation(M)).view(np.float64)
    elif kind == "equal":
        sc = np.full(M, 0.25)
    else:
        sc = np.where(rng.random(M) < 0.5, 0.25, -rng.uniform(0, 1, M))
        sc[rng.random(M) < 0.2] = np.nan
    out = torch.full((m,), -1, dtype=torch.int64, device="cuda:0")
    osc = torch.empty(m, dtype=torch.float64, device="cuda:0")
    cnt = B.sisso_topm(_d(sc), m, out, osc)
    fin = np.flatnonzero(np.isfinite(sc))
    order = fin[np.lexsort((fin, -sc[fin]))][:m]
    assert cnt == len(order)
    assert np.array_equal(out[:cnt].cpu().numpy(), order)
    np.testing.assert_array_equal(osc[:cnt].cpu().numpy(), sc[order])
