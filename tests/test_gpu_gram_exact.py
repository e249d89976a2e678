"""The FP64 Gram from residue products: exact on integer columns, and within
the rounding of its inputs on real ones, over the edges of its tiles (64, 128
and 256 features), K-steps (64 and 128 samples), sample chunks (65,536), task
padding and both finishing passes (up to 16 tasks together, more one by one)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
U = 2.0 ** -53


def gram(F, off):
    from paper_2502_20072_amd import L0Search
    y = np.linspace(-1.0, 2.0, F.shape[1])
    s = L0Search(F, y, off, D_max=1, k_max=1).gram()
    out = [s.gram_read(t)[0] for t in range(len(off) - 1)]
    s.close()
    return out


def integer_columns(rng, S, rows):
    """Small integers whose every task sums to zero: centring is exact, every
    cross product is an exact integer, and columns 0 and 1 of each task are
    orthogonal by construction."""
    F = np.zeros((S, sum(rows)))
    r0 = 0
    for n in rows:
        h = n // 2
        a = rng.integers(1, 9, size=(S, h)).astype(float)
        F[:, r0:r0 + h], F[:, r0 + h:r0 + 2 * h] = a, -a
        if S > 1:
            F[1, r0:r0 + 2 * h] = 0.0
            F[1, r0], F[1, r0 + h] = F[0, r0 + 1], F[0, r0 + 1]  # even part: orthogonal to the odd column 0
            F[1, r0 + 1], F[1, r0 + h + 1] = -F[0, r0 + 1], -F[0, r0 + 1]
        r0 += n
    return F


@pytest.mark.parametrize("S,rows", [
    (2, [4]), (63, [64]), (65, [66]), (127, [128]), (129, [130]), (257, [62]), (300, [1000]),
    (70, [66000]),                       # two chunks of samples
    (40, [64, 4, 130, 62]), (130, [200, 66]),
    (33, [6 + 2 * t for t in range(20)]),  # more than 16 tasks
    (20, [65600, 60]),                   # a task that starts in the second chunk
    (4097, [70]),                        # 256-wide tiles
])
def test_integer_columns_are_exact(S, rows):
    rng = np.random.default_rng(S + sum(rows))
    F = integer_columns(rng, S, rows)
    off = np.concatenate([[0], np.cumsum(rows)])
    pick = np.unique(np.concatenate([np.arange(min(S, 40)), rng.integers(0, S, 60), [S - 1]]))
    for t, G in enumerate(gram(F, off)):
        x = F[pick, off[t]:off[t + 1]]
        C = x @ x.T                      # exact: integers below 2^53
        d = np.sqrt(np.diag(C))
        # 1/sqrt(norm^2) is off by at most 2 U, its products and the result by U each
        ref = C / np.outer(d, d)
        got = G[np.ix_(pick, pick)]
        off_diag = ~np.eye(len(pick), dtype=bool)
        assert np.all(np.abs(got - ref)[off_diag] <= 10 * U * np.abs(ref)[off_diag])
        assert np.all(np.diag(G) == 1.0)
        assert np.array_equal(G, G.T)
        if S > 1:
            assert G[0, 1] == 0.0        # an exact zero stays one


@pytest.mark.parametrize("kind", ["gauss", "offset", "spike", "scale", "near"])
@pytest.mark.parametrize("S,rows", [(40, [100]), (64, [2000]), (30, [63, 129, 700]), (12, [66001])])
def test_real_columns(kind, S, rows):
    """Against 80-bit arithmetic.  Rounding of x - mean leaves at most 2 U of
    an entry (Cauchy-Schwarz), the norms (n / 64 + 7) U / 2 each, the scaling
    4 U; the integers' 2^-58 is below that."""
    n = sum(rows)
    rng = np.random.default_rng(S + n)
    F = rng.standard_normal((S, n))
    if kind == "offset":
        F += 100.0 * rng.standard_normal((S, 1))
    elif kind == "spike":
        F[::3, n // 2] = 1e4
    elif kind == "scale":
        F *= 10.0 ** rng.integers(-120, 120, (S, 1))
    elif kind == "near":
        F = F[:1] + 1e-6 * F
    off = np.concatenate([[0], np.cumsum(rows)])
    for t, G in enumerate(gram(F, off)):
        a, b = off[t], off[t + 1]
        x = F[:, a:b].astype(np.longdouble)
        # x - mean in double carries U |x|, which an offset or a spike makes
        # larger than U |x - mean|
        amp = float(max(1.0, np.max(np.sqrt((x * x).sum(1) / ((x - x.mean(1, keepdims=True)) ** 2).sum(1)))))
        x = x - x.mean(1, keepdims=True)
        x /= np.sqrt((x * x).sum(1, keepdims=True))
        ref = np.array([[(x[i] * x[j]).sum() for j in range(S)] for i in range(S)])
        err = np.abs((G - ref).astype(float))
        assert err.max() <= (2 * amp * (2 + (b - a) / 64 / 8) + (b - a) / 64 + 11) * U
        assert np.array_equal(G, G.T)


@pytest.mark.parametrize("S,rows", [
    (1, [4]), (63, [3]), (130, [5]), (300, [16]), (1000, [30]), (1300, [9]),   # few rows: FP64 products
    (129, [6, 21]), (600, [16, 33, 47]), (130, [5 + t % 3 for t in range(16)]),
    (70, [4 + t for t in range(17)]), (200, [9] * 64),
    (64, [600 + t for t in range(64)]),  # many long tasks of few features: FP64 products again
    (33, [5000] * 4), (200, [3000, 7]),  # parts of the samples, one of the tasks too short for them
    (260, [260] * 3), (257, [900] * 2),  # 128- and 256-wide tiles
])
def test_both_products(S, rows):
    """Either side of the line between the FP64 products and the residue ones,
    and the residue products' parts: within the rounding of FP64 sums (n / 2 U
    with the centring, whatever their order) of 80-bit arithmetic, unit diagonal,
    bitwise symmetric."""
    rng = np.random.default_rng(S + len(rows))
    off = np.concatenate([[0], np.cumsum(rows)])
    F = rng.standard_normal((S, off[-1])) + rng.standard_normal((S, 1))
    pick = np.unique(np.concatenate([np.arange(min(S, 20)), rng.integers(0, S, 30), [S - 1]]))
    for t, G in enumerate(gram(F, off)):
        x = F[:, off[t]:off[t + 1]].astype(np.longdouble)[pick]
        x = x - x.mean(1, keepdims=True)
        x /= np.sqrt((x * x).sum(1, keepdims=True))
        ref = (x @ x.T).astype(float)
        # x - mean carries U |x|; a task's columns of a few rows can be close to constant
        raw = F[pick, off[t]:off[t + 1]]
        amp = np.max(np.linalg.norm(raw, axis=1) / np.linalg.norm(raw - raw.mean(1, keepdims=True), axis=1))
        assert np.abs(G[np.ix_(pick, pick)] - ref).max() <= (rows[t] / 2 + 30) * amp * U
        assert np.all(np.diag(G) == 1.0) and np.array_equal(G, G.T)


def test_dead_and_non_finite_columns():
    """A constant column's row, column and diagonal are zero; a non-finite one
    is reported by the readout of a search."""
    from paper_2502_20072_amd import L0Search, SissoError
    rng = np.random.default_rng(5)
    F = rng.standard_normal((70, 150))
    F[3] = 2.5
    G = gram(F, [0, 150])[0]
    assert not G[3].any() and not G[:, 3].any()
    F[5, 7] = np.inf
    s = L0Search(F, rng.standard_normal(150), D_max=2, k_max=3).gram().search(2, 3)
    with pytest.raises(SissoError):
        s.topk()
    s.close()
