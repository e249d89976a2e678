"""The superset bound of the record-table searches on chained columns: a group
of four in which every column lies close to the span of the ones before it and
carries the direction that the last one added, so that each pivot is small but
usable and the inverse of the group's factor is large (squared norm up to
1e15).  On the CPU the bound's terms in double precision, against extended
precision, stay within half of the slacks for every base and column that the
search tries it on; on the GPU no search loses the best tuples."""
import math
import os
import re

import numpy as np
import pytest

import oracle
from synth.problems import Problem
from tests.parity import total_ss

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_20072_amd", "csrc",
                      "search.hip")


def constant(name):
    """A double constant of the search kernels' source."""
    return float(re.search(rf"\b{name} = ([0-9.e+-]+)", open(SOURCE).read()).group(1))


def chain(rng, q, pivots, weight):
    """Columns from the orthonormal rows of q: column m is close to row m - 1
    plus weight times earlier rows, and adds row m (its pivot)."""
    x = [q[0]]
    for m, p in enumerate(pivots, 1):
        v = q[m - 1] + weight * rng.standard_normal(m - 1) @ q[:m - 1]
        x.append(math.sqrt(1.0 - p) * v / np.linalg.norm(v) + math.sqrt(p) * q[m])
    return x


# ----------------------------------------------------------- the bound's terms
def terms(G, b, c, K, dtype):
    """The table of a base of K columns, and the terms of the bound for columns
    K (row j) and K + 1 (column k), batched over the first axis: the group's
    smallest pivot and |R^-1|^2, j's pivot, and p, d, zeta of the pair."""
    G, b, c = G.astype(dtype), b.astype(dtype), c.astype(dtype)
    B = len(G)
    L, Li, z = np.zeros((B, K, K), dtype), np.zeros((B, K, K), dtype), np.zeros((B, K), dtype)
    low, kappa, p = np.ones(B, dtype), np.zeros(B, dtype), c.copy()
    for m in range(K):
        d = np.ones(B, dtype)
        for l in range(m):
            s = G[:, l, m] - (L[:, m, :l] * L[:, l, :l]).sum(1)
            L[:, m, l] = s * Li[:, l, l]
            d -= L[:, m, l] ** 2
        low = np.minimum(low, d)
        Li[:, m, m] = 1 / np.sqrt(np.maximum(d, dtype(1e-30)))
        for l in range(m):
            Li[:, m, l] = -Li[:, m, m] * (L[:, m, l:m] * Li[:, l:m, l]).sum(1)
        z[:, m] = (Li[:, m, :m + 1] * b[:, :m + 1]).sum(1)
        p -= z[:, m] ** 2
        kappa += (Li[:, m, :m + 1] ** 2).sum(1)
    v = [np.stack([(Li[:, m, :m + 1] * G[:, :m + 1, x]).sum(1) for m in range(K)], 1) for x in (K, K + 1)]
    d = [1 - (w ** 2).sum(1) for w in v]
    e = [b[:, x] - (w * z).sum(1) for x, w in zip((K, K + 1), v)]
    zs = e[0] / d[0]
    u = G[:, K, K + 1] - (v[0] * v[1]).sum(1)
    return low, kappa, d[0], p - e[0] * zs, d[1] - u * u / d[0], e[1] - zs * u


@pytest.mark.parametrize("K", [4, 8])
def test_error_of_the_terms_within_half_the_slack(K):
    tau, slack = constant("S3_TAU"), constant("S3_SLACK")
    rng = np.random.default_rng(K)
    B = 6000
    G, b, c = np.empty((B, K + 2, K + 2)), np.empty((B, K + 2)), np.empty(B)
    for i in range(B):
        n = K + 3
        q = np.eye(n)
        low = 10.0 ** rng.uniform(-5.0, -1.0)
        x = chain(rng, q, np.maximum(tau, low * 10.0 ** rng.uniform(0.0, 1.5, K - 1)).clip(max=0.5),
                  10.0 ** rng.uniform(-2.0, 0.5))
        for own in (10.0 ** rng.uniform(-5.0, 0.0), 10.0 ** rng.uniform(-8.0, 0.0)):
            w = np.zeros(n)
            w[:len(x)] = rng.standard_normal(len(x)) * 10.0 ** -rng.uniform(0.0, 3.0, len(x))
            v = w / np.linalg.norm(w) + (x[K - 1] if rng.random() < 0.5 else 0.0)
            v = v / np.linalg.norm(v) + math.sqrt(own) * q[len(x)]
            x.append(v / np.linalg.norm(v))
        x = np.array(x)
        y = x.T @ (rng.standard_normal(K + 2) * 10.0 ** rng.uniform(-1.0, 2.0, K + 2))
        y = y / np.linalg.norm(y) + 10.0 ** -rng.uniform(1.0, 4.0) * q[K + 2]
        G[i], b[i], c[i] = x @ x.T, x @ y, y @ y
    at = np.arange(K + 2)
    G[:, at, at] = 1.0
    with np.errstate(all="ignore"):  # (bases with pivots of zero)
        low, kappa, dj, p, d, zeta = terms(G, b, c, K, np.float64)
        ref = terms(G, b, c, K, np.longdouble)
    # the rule of the search: the base's pivots, then a smallest pivot of j
    room = np.sqrt(slack / (4 * K * (K + 1) * 2.0 ** -53 * kappa)) - 1.0
    used = (low > tau) & (room >= 1.0) & (dj > np.maximum(tau, 1.0 / np.maximum(room, 1e-30) ** 2)) & (ref[4] > 0)
    assert used.sum() > B // 50 and kappa[used].max() > 1e3
    err = np.stack([np.abs(p - ref[3]) / c, np.abs(d - ref[4]), np.abs(zeta - ref[5]) / np.sqrt(c)])
    assert float(err[:, used].max()) <= slack / 2
    # and the rule is needed: among the other bases with the same pivots it is larger
    assert float(err[:, (low > tau) & (dj > tau) & ~used & (ref[4] > 0)].max()) > slack


# ------------------------------------------------------------------ searches
def chained_problem(seed, S, T):
    """Columns 0 to 3 chained, 4 close to 3, and from 8 on copies (1e-5 apart)
    of a column in the span of 3 and 4 but for 2e-4 of its own.  y is 3 and 4 and
    what column 8 adds to them: the tuples (3, 4, k), k >= 8, are the best and
    have pivots above 1e-8, and the pre-pass finds enough of them for its bound."""
    rng = np.random.default_rng(seed)
    n, phi = 120, rng.uniform(0.5, 1.5)

    def unit(m):
        d = rng.standard_normal((m, n))
        d -= d.mean(1, keepdims=True)
        return d / np.linalg.norm(d, axis=1, keepdims=True)

    F, y = np.empty((S, n * T)), np.empty(n * T)
    for t in range(T):
        q = np.linalg.qr(np.c_[np.ones(n), rng.standard_normal((n, 6))])[0][:, 1:].T
        f = unit(S)
        f[:4] = chain(np.random.default_rng([seed, 1]), q, (1.2e-5, 1.3e-5, 5e-5), 0.2)
        f[4] = math.sqrt(1.0 - 1.3e-5) * f[3] + math.sqrt(1.3e-5) * q[4]
        f[8:] = math.cos(phi) * f[3] + math.sin(phi) * q[4] + 2e-4 * q[5] + 1e-5 * f[8:]
        r = f[8] - f[[3, 4]].T @ np.linalg.lstsq(f[[3, 4]].T, f[8], rcond=None)[0]
        s = slice(n * t, n * t + n)
        y[s] = (1.0 + 0.2 * t) * (3.0 * f[3] + 0.5 * q[4] + r / np.linalg.norm(r)) + math.sqrt(3e-7) * unit(1)[0]
        F[:, s] = f
    return Problem(F, y, np.arange(T + 1, dtype=np.int64) * n, [3, 4, 8], 3, 20, [], {})


SEEDS = range(24)


def check(p, D, k, idx, sse):
    """The returned tuples are the oracle's k best.  A tuple's pivots go down to
    4e-8 and 1.3e-5 here, so its coefficients reach b = 1e6 |y| and the
    normal equations leave (2^-53 b)^2 / (4e-8 * 1.3e-5) = 2e-8 c per unit of
    their constant on its SSE: 1e-5 c is taken for both (the tuples without
    columns 3 and 4 miss y by c / 10)."""
    tol = 1e-5 * total_ss(p)
    best, ref, _ = oracle.topk(p.F, p.y, D, k, p.task_offsets)
    got = [tuple(int(v) for v in t) for t in idx]
    assert len(set(got)) == k
    for t, s in zip(got, sse):
        assert abs(s - oracle.tuple_sse(p.F, p.y, t, p.task_offsets)) <= tol
        assert s <= ref[-1] + 2 * tol, (t, s, ref[-1])
    for t, s in zip(best, ref):
        assert tuple(int(v) for v in t) in got or s >= ref[-1] - 2 * tol, (t, s)


def run(p, D, k):
    from paper_2502_20072_amd import L0Search
    s = L0Search(p.F, p.y, p.task_offsets, D_max=D, k_max=k)
    out = s.gram().search(D, k).topk()
    s.close()
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("T", [1, 2])
@pytest.mark.parametrize("seed", SEEDS)
def test_d3(seed, T):
    p = chained_problem(seed, 88, T)
    idx, sse, _ = run(p, 3, 20)
    check(p, 3, 20, idx, sse)


@pytest.mark.gpu
@pytest.mark.parametrize("seed", SEEDS)
def test_d4(seed):
    p = chained_problem(seed, 30, 1)
    idx, sse, _ = run(p, 4, 15)
    check(p, 4, 15, idx, sse)


@pytest.mark.gpu
def test_batch():
    from paper_2502_20072_amd import L0Search
    from paper_2502_20072_amd import _binding as B
    ps = [chained_problem(seed, 88, 1) for seed in SEEDS]
    hs = [L0Search(p.F, p.y, p.task_offsets, D_max=3, k_max=20) for p in ps]
    b = B.sisso_l0_batch_create([h.handle for h in hs], 3, 20)
    B.sisso_l0_batch_launch(b)
    try:
        for p, h in zip(ps, hs):
            h.last_D, h.last_k = 3, 20
            idx, sse, _ = h.topk()
            check(p, 3, 20, idx, sse)
    finally:
        B.sisso_l0_batch_destroy(b)
        for h in hs:
            h.close()

