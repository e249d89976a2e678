"""Performance cases of the library: the calls a SISSO user's program makes,
through the public entry points, at the sizes of this repository's own
workloads and over the ranges around them.

A case is a dict of plain values with a ``kind``:

* ``l0``      one subspace: Gram, exhaustive search of all D-tuples, readout
              of the k best models (``L0Search``);
* ``batch``   many independent subspaces in one captured graph
              (``sisso_l0_batch_*``), every result read out;
* ``screen``  one screening pass over a rung of features created on the fly
              from stored children, against several residuals, and the exact
              top-m (``SisScreen.score_op``, ``sisso_topm``);
* ``fit``     the whole dimension loop over stored candidate features
              (``sisso_fit``: screening, search, residuals, D = 1..3);
* ``propose`` the learned proposal at D = 4: Gram, then two-stage scoring of
              prefixes by the network and the exact search of the best ones
              (``learned.propose_two_stage``);
* ``train``   one training step of the proposal network: forward, backward,
              Adam (``sisso_mlp_*``).

Inputs are synthetic and drawn on the GPU from the seed.  ``trees`` columns
are random operator trees of rung 1-2 over ten lognormal primary features,
duplicates dropped, standardised; ``factor`` columns share 20 latent factors
(used where the subspace is too large for a duplicate filter).  The target is
a linear combination of D of the columns plus noise, per task its own
coefficients.
"""
import math

import numpy as np
import torch

from paper_2502_20072_amd import L0Search
from paper_2502_20072_amd import _binding as B
from paper_2502_20072_amd import learned

DEV = "cuda:0"
BETA = (1.5, -0.8, 0.6, -0.4)
BINARY = ("add", "sub", "mul", "div", "abs_diff")
PRECISIONS = {"fp64": B.SISSO_PREC_FP64, "bf16": B.SISSO_PREC_BF16_COMP, "fp16": B.SISSO_PREC_FP16_COMP,
              "fp32": B.SISSO_PREC_FP32_SOLVE}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest search a user makes: a first look at a small data set,
        # where launches and the readout are the cost
        dict(name="l0_n100_s200_d2", kind="l0", rows="100", S=200, D=2, k=10, sigma=0.01, gen="trees", prec="fp64"),
        # the ordinary descriptor search (the benchmark's default workload)
        dict(name="l0_n2000_s1000_d3", kind="l0", rows="2000", S=1000, D=3, k=100, sigma=0.05, gen="trees",
             prec="fp64"),
        # multi-task: 16 ragged tasks (materials classes with 53 to 3111 rows),
        # one descriptor, coefficients per task
        dict(name="l0_t16_s1500_d3", kind="l0",
             rows="1289,333,66,1532,59,53,211,97,402,739,151,3111,78,618,125,823", S=1500, D=3, k=100, sigma=0.05,
             gen="trees", prec="fp64"),
        # the largest descriptor dimension
        dict(name="l0_n2000_s600_d4", kind="l0", rows="2000", S=600, D=4, k=100, sigma=0.05, gen="trees",
             prec="fp64"),
        # many samples: the Gram dominates
        dict(name="l0_n50000_s4096_d2", kind="l0", rows="50000", S=4096, D=2, k=100, sigma=0.05, gen="trees",
             prec="fp64"),
        # the same data with the reduced-precision Gram a user picks for speed
        dict(name="l0_n50000_s4096_d2_fp16", kind="l0", rows="50000", S=4096, D=2, k=100, sigma=0.05, gen="trees",
             prec="fp16"),
        # the largest subspace: 50,000 features kept by the screening, pairs
        dict(name="l0_n2400_s50000_d2", kind="l0", rows="2400", S=50000, D=2, k=100, sigma=0.05, gen="factor",
             prec="fp64"),
        # a parameter scan: 64 subspaces of different sizes in one launch
        dict(name="batch64_d3", kind="batch", P=64, S_lo=200, S_hi=2000, n_lo=100, n_hi=5000, D=3, k=100,
             sigma=0.05),
        # one screening pass over a created rung: five operators on every
        # child pair, ten residuals, the 1000 best kept
        dict(name="screen_s1000_n2000", kind="screen", children=1000, rows="2000", nres=10, m=1000, ops="all"),
        # the whole dimension loop over stored candidates, two tasks
        dict(name="fit_m300000_n1013", kind="fit", M=300000, rows="600,413", D=3, m_sis=100, n_res=10, k=10),
        # the learned proposal in use
        dict(name="propose_s600_d4", kind="propose", rows="2000", S=600, D=4, k=100, sigma=0.05, budget=1e-4),
        # the learned proposal in training: one step of the fit's batch size
        dict(name="train_b4096", kind="train", n=4096, lr=2e-3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_rows(rng, T, lo, hi):
    return ",".join(str(_log_int(rng, lo, hi)) for _ in range(T))


def draw(rng):
    kind = rng.choice(["l0"] * 7 + ["batch", "screen", "fit", "propose", "train"])
    if kind == "l0":
        D = rng.choice([2, 2, 3, 3, 3, 4])
        T = rng.choice([1, 1, 1, 2, rng.randint(3, 16)])
        sigma = round(math.exp(rng.uniform(math.log(0.01), math.log(0.5))), 4)
        k = rng.choice([1, 10, 100, 100])
        prec = rng.choice(["fp64"] * 6 + ["bf16", "fp16", "fp32"])
        if T == 1:
            n = _log_int(rng, 100, 50000)
            rows = str(n)
        else:
            rows = _draw_rows(rng, T, 60, 3000)
            n = sum(int(r) for r in rows.split(","))
        if D == 2:
            S = _log_int(rng, 200, 12000)
        elif D == 3:
            S = _log_int(rng, 200, 5000 if T <= 2 and prec != "fp32" else 1500)
        else:
            S = _log_int(rng, 100, 600 if T == 1 else 200)
        while n * S * S > 50000 * 4096 * 4096 or S * S * T > 16 * 2000 * 2000 * 8:
            S = S * 3 // 4
        return dict(kind="l0", rows=rows, S=S, D=D, k=k, sigma=sigma, gen="trees" if S <= 6000 else "factor",
                    prec=prec)
    if kind == "batch":
        S_hi = _log_int(rng, 300, 2000)
        return dict(kind="batch", P=rng.randint(3, 40), S_lo=rng.randint(150, S_hi), S_hi=S_hi, n_lo=100,
                    n_hi=_log_int(rng, 300, 5000), D=3, k=rng.choice([10, 100]), sigma=0.05)
    if kind == "screen":
        T = rng.choice([1, 1, 2, 3])
        rows = _draw_rows(rng, T, 70, 2000 // T)
        return dict(kind="screen", children=_log_int(rng, 60, 1000), rows=rows, nres=rng.choice([1, 3, 5, 10, 10, 16]),
                    m=rng.choice([100, 500, 1000]), ops=rng.choice(["all", "add,mul", "sub,div", "mul,abs_diff"]))
    if kind == "fit":
        T = rng.choice([1, 2])
        return dict(kind="fit", M=_log_int(rng, 5000, 300000), rows=_draw_rows(rng, T, 80, 1013 // T),
                    D=rng.choice([2, 3]), m_sis=rng.randint(20, 100), n_res=rng.randint(1, 10), k=10)
    if kind == "propose":
        return dict(kind="propose", rows=str(_log_int(rng, 200, 2000)), S=rng.randint(150, 600), D=rng.choice([3, 4]),
                    k=100, sigma=0.05, budget=rng.choice([1e-3, 1e-4]))
    return dict(kind="train", n=_log_int(rng, 200, 16384), lr=2e-3)


# --------------------------------------------------------------------- inputs
def _rows(case):
    return [int(r) for r in str(case["rows"]).split(",")]


def _offsets(case):
    return np.concatenate([[0], np.cumsum(_rows(case))]).astype(np.int64)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _randint(g, hi, n):
    return torch.randint(0, hi, (n,), generator=g, device=DEV)


def _op(op, a, b):
    """The ten tree operators, op[i] applied to rows a[i], b[i]."""
    fns = (lambda x, y: x + y, lambda x, y: x - y, lambda x, y: x * y, lambda x, y: x / y,
           lambda x, y: (x - y).abs(), lambda x, y: x.exp(), lambda x, y: x.log(), lambda x, y: x.sqrt(),
           lambda x, y: x * x, lambda x, y: x * x * x)
    out = torch.empty_like(a)
    for i, f in enumerate(fns):
        sel = (op == i).nonzero()[:, 0]
        if sel.numel():
            out[sel] = f(a[sel], b[sel])
    return out


def _eval_trees(prim, t, sel):
    r1 = _op(t["op1"][sel], prim[t["i1"][sel]], prim[t["j1"][sel]])
    two = t["rung2"][sel][:, None]
    r1b = _op(t["op1b"][sel], prim[t["i1b"][sel]], prim[t["j1b"][sel]])
    other = torch.where(t["leaf"][sel][:, None], prim[t["i2"][sel]], r1b)
    sw = t["swap"][sel][:, None]
    r2 = _op(t["op2"][sel], torch.where(sw, other, r1), torch.where(sw, r1, other))
    return torch.where(two, r2, r1)


def _standard(F):
    F = F - F.mean(1, keepdim=True)
    return (F / F.std(1, keepdim=True, unbiased=False)).contiguous()


def _tree_columns(g, n, S):
    """S random operator trees over ten lognormal primaries: non-finite,
    constant and duplicate (|r| > 0.9999) columns dropped."""
    prim = (0.5 * _randn(g, 10, n)).exp()
    N = 4 * S + 2000
    t = {q: _randint(g, 10, N) for q in ("op1", "i1", "op1b", "i1b", "op2", "i2")}
    t["j1"] = (t["i1"] + 1 + _randint(g, 9, N)) % 10
    t["j1b"] = (t["i1b"] + 1 + _randint(g, 9, N)) % 10
    for q in ("rung2", "leaf", "swap"):
        t[q] = _randint(g, 2, N) == 1
    # the filter on the first rows, then the survivors on all of them
    m = min(n, 512)
    keep = torch.arange(N, device=DEV)
    head = _eval_trees(prim[:, :m].contiguous(), t, keep)
    head = torch.cat([prim[:, :m], head])
    x = head - head.mean(1, keepdim=True)
    nrm = x.norm(dim=1, keepdim=True)
    fine = torch.isfinite(nrm[:, 0]) & (nrm[:, 0] > 1e-9 * head.abs().amax(1)) & (head.abs().amax(1) < 1e8)
    x = torch.where(fine[:, None], x / nrm, torch.zeros_like(x))
    dup = torch.zeros(N + 10, dtype=torch.bool, device=DEV)
    for a in range(0, N + 10, 4096):
        r = (x[a:a + 4096] @ x[:a + 4096].T).abs() > 0.9999
        r &= torch.arange(r.shape[1], device=DEV)[None] < torch.arange(a, a + r.shape[0], device=DEV)[:, None]
        dup[a:a + 4096] = r.any(1)
    ids = (fine & ~dup).nonzero()[:, 0]
    ids = ids[:S + S // 8 + 64]
    F = torch.cat([prim, _eval_trees(prim, t, ids[ids >= 10] - 10)])
    big = F.abs().amax(1)
    F = F[torch.isfinite(big) & (big < 1e9)][:S]
    if F.shape[0] < S:
        raise RuntimeError("too few distinct columns for S = %d, n = %d" % (S, n))
    return _standard(F)


def _factor_columns(g, n, S):
    z = _randn(g, 20, n)
    F = torch.empty(S, n, dtype=torch.float64, device=DEV)
    for a in range(0, S, 8192):
        b = min(S, a + 8192)
        F[a:b] = _standard(_randn(g, b - a, 20) @ z + _randn(g, b - a, n))
    return F


def _problem(g, rows, S, D, sigma, gen):
    n = sum(rows)
    F = (_tree_columns if gen == "trees" else _factor_columns)(g, n, S)
    planted = torch.randperm(S, generator=g, device=DEV)[:D]
    y = sigma * _randn(g, n)
    beta = torch.tensor(BETA[:D], dtype=torch.float64, device=DEV)
    r0 = 0
    for r in rows:
        b, a = beta, 0.0
        if len(rows) > 1:
            b = beta * (1.0 + 0.25 * _randn(g, D))
            a = 2.0 * torch.rand(1, generator=g, device=DEV, dtype=torch.float64) - 1.0
        y[r0:r0 + r] += a + b @ F[planted, r0:r0 + r]
        r0 += r
    return F, y


def _batch_sizes(case):
    rng = np.random.default_rng(case["P"] * 1000003 + case["S_hi"] * 101 + case["n_hi"])
    return [(int(rng.integers(case["S_lo"], case["S_hi"] + 1)), int(rng.integers(case["n_lo"], case["n_hi"] + 1)))
            for _ in range(case["P"])]


def _children(g, case):
    """Children and residuals of a screening pass: row 0 the target, the
    others residuals of earlier models."""
    n = sum(_rows(case))
    X = _tree_columns(g, n, case["children"])
    p = torch.randperm(case["children"], generator=g, device=DEV)[:3]
    y = 1.5 * X[p[0]] * X[p[1]] - 0.8 * X[p[2]] + 0.05 * _randn(g, n)
    R = y[None] + 0.3 * _randn(g, case["nres"], n)
    R[0] = y
    pairs = torch.triu_indices(case["children"], case["children"], 1, device=DEV).T.to(torch.int32).contiguous()
    return X, R.contiguous(), pairs


def _ops(case):
    return BINARY if case["ops"] == "all" else tuple(case["ops"].split(","))


def _candidates(g, case):
    """Stored candidates of a dimension loop: products, ratios and absolute
    differences of pairs of positive columns, standardised."""
    n, M = sum(_rows(case)), case["M"]
    c = int(math.ceil(0.5 + math.sqrt(0.25 + 2.0 * M / 3.0))) + 1
    P = (0.5 * _randn(g, c, n)).exp()
    pr = torch.triu_indices(c, c, 1, device=DEV)
    X = torch.empty(M, n, dtype=torch.float64, device=DEV)
    per = (M + 2) // 3
    for q in range(3):
        for a in range(q * per, min(M, (q + 1) * per), 65536):
            b = min(M, (q + 1) * per, a + 65536)
            u, v = P[pr[0, a - q * per:b - q * per]], P[pr[1, a - q * per:b - q * per]]
            X[a:b] = _standard(u * v if q == 0 else u / v if q == 1 else (u - v).abs())
    pick = torch.randperm(M, generator=g, device=DEV)[:case["D"]]
    y = 0.3 * _randn(g, n)
    r0 = 0
    for r in _rows(case):
        b = torch.tensor(BETA[:case["D"]], dtype=torch.float64, device=DEV) * (1.0 + 0.25 * _randn(g, case["D"]))
        y[r0:r0 + r] += b @ X[pick, r0:r0 + r]
        r0 += r
    return X, y


class _Batch:
    """The handles of a batch and its captured graph."""

    def __init__(self, searches, D, k):
        self.searches, self.D, self.k = searches, D, k
        self.batch = B.sisso_l0_batch_create([s.handle for s in searches], D, k)
        for s in searches:
            s.last_D, s.last_k = D, k

    def __del__(self):
        if getattr(self, "batch", None):
            B.sisso_l0_batch_destroy(self.batch)


def _net(seed):
    """A proposal network that ranks prefixes mostly by their own fit, as a
    trained one does: small random layers and one strong path from the first
    input (the prefix's R^2) to the output."""
    net = learned.ProposalNet(seed=int(seed) % 100003, device=DEV)
    I, H = B.MLP_IN, B.MLP_HIDDEN
    net.params *= 0.1
    for at, v in ((0, 2.0), (I * H + H, 4.0), (I * H + H + H * H + H, 4.0)):  # W1[0, 0], W2[0, 0], W3[0]
        net.params[at] = v
    return net


def prepare(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "l0":
        F, y = _problem(g, _rows(case), case["S"], case["D"], case["sigma"], case["gen"])
        return dict(case=case, s=L0Search(F, y, _offsets(case), D_max=case["D"], k_max=case["k"],
                                          precision=PRECISIONS[case["prec"]]))
    if kind == "batch":
        searches = []
        for S, n in _batch_sizes(case):
            F, y = _problem(g, [n], S, case["D"], case["sigma"], "trees")
            searches.append(L0Search(F, y, [0, n], D_max=case["D"], k_max=case["k"]))
        return dict(case=case, b=_Batch(searches, case["D"], case["k"]))
    if kind == "screen":
        X, R, pairs = _children(g, case)
        M = pairs.shape[0] * len(_ops(case))
        return dict(case=case, X=X, pairs=pairs, h=B.SisScreen(R, _offsets(case)),
                    scores=torch.empty(M, dtype=torch.float64, device=DEV),
                    valid=torch.empty(M, dtype=torch.uint8, device=DEV),
                    idx=torch.zeros(case["m"], dtype=torch.int64, device=DEV),
                    best=torch.zeros(case["m"], dtype=torch.float64, device=DEV))
    if kind == "fit":
        X, y = _candidates(g, case)
        return dict(case=case, X=X, y=y)
    if kind == "propose":
        F, y = _problem(g, _rows(case), case["S"], case["D"], case["sigma"], "trees")
        return dict(case=case, s=L0Search(F, y, _offsets(case), D_max=case["D"], k_max=case["k"]), net=_net(seed))
    net = learned.ProposalNet(seed=int(seed) % 100003, device=DEV)
    n, f32 = case["n"], dict(dtype=torch.float32, device=DEV)
    # prefix features: fits and correlations in [0, 1], and 1/m; targets are
    # -log10 of unexplained fractions.  The moments are those of a run that
    # is under way (a first step from zero moments happens once).
    x = torch.rand(n, B.MLP_IN, generator=g, **f32)
    x[:, 7] = torch.where(torch.rand(n, generator=g, **f32) < 0.5, 0.5, 1.0 / 3.0)
    t = 2.0 * x[:, 0] + 0.2 * torch.rand(n, generator=g, **f32)
    m = 1e-3 * torch.randn(B.MLP_NPARAM, generator=g, **f32)
    v = 1e-5 * (0.5 + torch.rand(B.MLP_NPARAM, generator=g, **f32))
    return dict(case=case, p=net.params, x=x.contiguous(), t=t.contiguous(), m=m, v=v, step=100,
                out=torch.empty(n, **f32), grad=torch.empty(B.MLP_NPARAM, **f32), loss=torch.empty(1, **f32),
                ws=torch.empty(B.sisso_mlp_workspace_bytes(n), dtype=torch.uint8, device=DEV))


# ------------------------------------------------------------------- one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "l0":
        s = state["s"]
        idx, sse, coef = s.gram().search(case["D"], case["k"]).topk()
        return dict(idx=idx, sse=sse, coef=coef)
    if kind == "batch":
        b = state["b"]
        B.sisso_l0_batch_launch(b.batch)
        got = [s.topk() for s in b.searches]
        return dict(idx=np.stack([q[0] for q in got]), sse=np.stack([q[1] for q in got]),
                    coef=np.stack([q[2] for q in got]))
    if kind == "screen":
        X, pairs, sc, va = state["X"], state["pairs"], state["scores"], state["valid"]
        P = pairs.shape[0]
        for o, op in enumerate(_ops(case)):
            state["h"].score_op(op, X, pairs, 1e-5, 1e8, sc[o * P:(o + 1) * P], va[o * P:(o + 1) * P])
        cnt = B.sisso_topm(sc, case["m"], state["idx"], state["best"])
        return dict(scores=sc, valid=va, idx=state["idx"], best=state["best"], count=cnt)
    if kind == "fit":
        return B.sisso_fit(state["X"], state["y"], _offsets(case), case["D"], case["m_sis"], case["n_res"], case["k"])
    if kind == "propose":
        s = state["s"]
        s.gram()
        learned.propose_two_stage(s, case["D"], case["k"], state["net"].predict, budget_frac=case["budget"])
        idx, sse, coef = s.topk()
        return dict(idx=idx, sse=sse, coef=coef)
    st = torch.cuda.current_stream().cuda_stream
    B.sisso_mlp_forward(state["p"], state["x"], state["out"], state["ws"], st)
    B.sisso_mlp_backward(state["p"], state["x"], state["t"], state["grad"], state["loss"], state["ws"], st)
    B.sisso_mlp_adam(state["p"], state["grad"], state["m"], state["v"], state["step"], case["lr"], st)
    return dict(out=state["out"], grad=state["grad"], loss=state["loss"], params=state["p"], m=state["m"],
                v=state["v"])


# ----------------------------------------------------------------- least work
def _l0_flops(n, S, D, T):
    # the symmetric Gram once, then per tuple and task the solve of the last
    # index against a hoisted prefix (an FMA counts two)
    return float(n) * S * (S + 1) + 4.0 * n * S + float(math.comb(S, D)) * T * (2 * (D - 2) + 7)


def work(case):
    kind = case["kind"]
    if kind == "l0":
        rows, S, D, k = _rows(case), case["S"], case["D"], case["k"]
        n, T = sum(rows), len(_rows(case))
        return dict(bytes=8.0 * n * (S + 1) + k * (8.0 + 4 * D + 8 * T * (D + 1)), flops=_l0_flops(n, S, D, T))
    if kind == "batch":
        out = 8.0 + 4 * case["D"] + 8 * (case["D"] + 1)
        return dict(bytes=sum(8.0 * n * (S + 1) + case["k"] * out for S, n in _batch_sizes(case)),
                    flops=sum(_l0_flops(n, S, case["D"], 1) for S, n in _batch_sizes(case)))
    if kind == "screen":
        n, c = sum(_rows(case)), case["children"]
        P = math.comb(c, 2) * len(_ops(case))
        return dict(bytes=8.0 * n * (c + case["nres"]) + 8.0 * math.comb(c, 2) + 9.0 * P + 16.0 * case["m"],
                    flops=float(P) * n * (7 + 2 * case["nres"]))
    if kind == "fit":
        n, M, D, m = sum(_rows(case)), case["M"], case["D"], case["m_sis"]
        # every dimension screens all candidates against its residuals
        passes = [1] + [case["n_res"]] * (D - 1)
        return dict(bytes=D * 8.0 * n * M, flops=sum(float(M) * n * (6 + 2 * r) for r in passes) +
                    sum(_l0_flops(n, d * m, d, len(_rows(case))) for d in range(1, D + 1)))
    if kind == "propose":
        n, S, D = sum(_rows(case)), case["S"], case["D"]
        tuples = case["budget"] * math.comb(S, D)
        first = math.comb(S, D - 2)
        kept = max(256.0, 32.0 * tuples / (S - D + 1) / (S - D + 2))
        scored = first + kept * (S - D + 2)
        return dict(bytes=8.0 * n * (S + 1) + case["k"] * (16.0 + 4 * D + 8 * D),
                    flops=float(n) * S * (S + 1) + scored * 2.0 * (8 * 128 + 128 * 128 + 128) +
                    tuples * (2 * (D - 2) + 7))
    n = case["n"]
    per = 8 * 128 + 128 * 128 + 128
    return dict(bytes=4.0 * (n * (B.MLP_IN + 2) + 8 * B.MLP_NPARAM), flops=6.0 * n * per)


# ------------------------------------------------------------ 64-bit reference
def _centred(F, y, offs):
    """Per task: centred columns scaled to unit norm, centred target."""
    out = []
    for a, b in zip(offs[:-1], offs[1:]):
        x = F[:, a:b] - F[:, a:b].mean(1, keepdim=True)
        nrm = x.norm(dim=1, keepdim=True)
        live = nrm[:, 0] ** 2 > 1e-10 * F[:, a:b].square().sum(1)
        x = torch.where(live[:, None], x / nrm, torch.zeros_like(x))
        yc = y[a:b] - y[a:b].mean()
        out.append((x, yc))
    return out


def _keep_best(best, sse, tup, keep):
    """Merge new (sse, tuples) into the running list of the best."""
    s, t = torch.cat([best[0], sse]), torch.cat([best[1], tup])
    o = torch.argsort(s)[:keep]
    return s[o], t[o]


def _best_tuples(cols, S, D, keep):
    """The `keep` tuples of least SSE (summed over tasks), by normal equations
    in 64 bits, slice by slice of the first index."""
    G = [x @ x.T for x, _ in cols]
    b = [x @ yc for x, yc in cols]
    c = [yc @ yc for _, yc in cols]
    inf = float("inf")
    best = (torch.empty(0, dtype=torch.float64, device=DEV), torch.empty(0, D, dtype=torch.int64, device=DEV))
    ar = torch.arange(S, device=DEV)

    def take(sse, make):
        nonlocal best
        cut = best[0][-1] if best[0].numel() >= keep else torch.tensor(inf, device=DEV, dtype=torch.float64)
        flat = sse.reshape(-1)
        hit = (flat < cut).nonzero()[:, 0]
        if hit.numel() > 4 * keep:
            top = torch.topk(flat[hit], keep, largest=False).indices
            hit = hit[top]
        if hit.numel():
            best = _keep_best(best, flat[hit], make(hit), keep)

    if D == 1:
        sse = sum(cc - bb * bb for cc, bb in zip(c, b))
        return _keep_best(best, sse, ar[:, None], keep)
    for i in range(S - D + 1):
        lo = i + 1
        m = S - lo
        tot = 0.0
        for g, bb, cc in zip(G, b, c):
            gi = g[i, lo:]
            z0 = bb[i]
            d1 = g.diagonal()[lo:] - gi * gi           # pivots of the second index
            e1 = bb[lo:] - gi * z0
            ok1 = d1 > 1e-10
            p = torch.where(ok1 & (g[i, i] > 0.5), cc - z0 * z0 - e1 * e1 / d1, torch.full_like(d1, inf))
            if D == 2:
                tot = tot + p
                continue
            u = g[lo:, lo:] - gi[:, None] * gi[None]
            al = torch.where(ok1, 1.0 / d1, torch.zeros_like(d1))
            if D == 3:
                d2 = d1[None] - u * u * al[:, None]
                z = e1[None] - u * (e1 * al)[:, None]
                sse = torch.where(d2 > 1e-10, p[:, None] - z * z / d2, inf)
                tot = tot + sse
                continue
            # D = 4: the second index j, then (third, fourth)
            tot = tot if torch.is_tensor(tot) else torch.zeros(m, m, m, dtype=torch.float64, device=DEV)
            w = u * al.sqrt()[:, None]                   # (j, x)
            d2 = d1[None] - w * w
            e2 = e1[None] - w * (e1 * al.sqrt())[:, None]
            ok2 = d2 > 1e-10
            al2 = torch.where(ok2, 1.0 / d2, torch.zeros_like(d2))
            p2 = torch.where(ok2 & torch.isfinite(p)[:, None], p[:, None] - e2 * e2 * al2, inf)
            q = u[None] - w[:, :, None] * w[:, None, :]  # (j, x, k)
            d3 = d2[:, None, :] - q * q * al2[:, :, None]
            z = e2[:, None, :] - q * (e2 * al2)[:, :, None]
            tot += torch.where(d3 > 1e-10, p2[:, :, None] - z * z / d3, inf)
            del q, d3, z
        if D == 2:
            take(tot, lambda h: torch.stack([torch.full_like(h, i), lo + h], 1))
        elif D == 3:
            tot = torch.where(ar[:m, None] < ar[None, :m], tot, inf)
            take(tot, lambda h: torch.stack([torch.full_like(h, i), lo + h // m, lo + h % m], 1))
        else:
            tri = (ar[:m, None, None] < ar[None, :m, None]) & (ar[None, :m, None] < ar[None, None, :m])
            tot = torch.where(tri, tot, inf)
            take(tot, lambda h: torch.stack([torch.full_like(h, i), lo + h // (m * m), lo + h // m % m, lo + h % m],
                                            1))
    return best


def _direct_sse(F, y, offs, tup):
    """SSE of each tuple's fit from the columns themselves (QR, per task)."""
    tot = torch.zeros(tup.shape[0], dtype=torch.float64, device=DEV)
    for a, b in zip(offs[:-1], offs[1:]):
        A = F[:, a:b][tup]                               # (q, D, n)
        A = A - A.mean(2, keepdim=True)
        yc = y[a:b] - y[a:b].mean()
        r = yc.expand(A.shape[0], -1).clone()
        for _ in range(2):                               # orthonormalise and project, twice
            Q = torch.empty_like(A)
            for d in range(A.shape[1]):
                v = A[:, d].clone()
                for _ in range(2):
                    for e in range(d):
                        v = v - (Q[:, e] * v).sum(1, keepdim=True) * Q[:, e]
                Q[:, d] = v / v.norm(dim=1, keepdim=True)
            for d in range(A.shape[1]):
                r = r - (Q[:, d] * r).sum(1, keepdim=True) * Q[:, d]
        tot += r.square().sum(1)
    return tot


def _exact_models(F, y, offs, D, k):
    s, t = _best_tuples(_centred(F, y, offs), F.shape[0], D, 2 * k + 64)
    ok = torch.isfinite(s)
    t = t[ok]
    sse = _direct_sse(F, y, offs, t)
    o = torch.argsort(sse)[:k]
    return sse[o], t[o]


def _exact_scores(cols, R, offs):
    """SIS scores of columns (M, n) against residuals R (nres, n)."""
    num, tot = 0.0, 0.0
    flat = torch.zeros(cols.shape[0], dtype=torch.bool, device=DEV)
    for a, b in zip(offs[:-1], offs[1:]):
        x = cols[:, a:b]
        xc = x - x.mean(1, keepdim=True)
        xss = xc.square().sum(1)
        flat |= ~(xss > 1e-10 * x.square().sum(1))
        rc = R[:, a:b] - R[:, a:b].mean(1, keepdim=True)
        num = num + (xc @ rc.T).square() / xss[:, None]
        tot = tot + rc.square().sum(1)
    s = (num / tot[None]).amax(1)
    return torch.where(flat, torch.full_like(s, float("nan")), s)


def exact(case, seed):
    g = _gen(seed)
    kind = case["kind"]
    if kind == "l0":
        offs = _offsets(case)
        F, y = _problem(g, _rows(case), case["S"], case["D"], case["sigma"], case["gen"])
        if math.comb(case["S"], case["D"]) * len(_rows(case)) > 1.2e10:
            return None
        sse, _ = _exact_models(F, y, offs, case["D"], case["k"])
        return dict(idx=None, sse=sse, coef=None)
    if kind == "batch":
        out = []
        for S, n in _batch_sizes(case):
            F, y = _problem(g, [n], S, case["D"], case["sigma"], "trees")
            if len(out) == 0 and case["P"] * case["S_hi"] > 40000:
                return None  # thousands of slices: over 20 seconds
            out.append(_exact_models(F, y, [0, n], case["D"], case["k"])[0])
        return dict(idx=None, sse=torch.stack(out), coef=None)
    if kind == "screen":
        X, R, pairs = _children(g, case)
        offs, per, scores = _offsets(case), pairs.shape[0], []
        step = max(1, 40_000_000 // X.shape[1])
        for op in _ops(case):
            for a in range(0, per, step):
                u, v = X[pairs[a:a + step, 0].long()], X[pairs[a:a + step, 1].long()]
                v = _op(torch.full((u.shape[0],), BINARY.index(op), device=DEV), u, v)
                mx = v.abs().amax(1)
                s = _exact_scores(v, R, offs)
                bad = ~torch.isfinite(mx) | (mx < 1e-5) | (mx > 1e8)
                scores.append(torch.where(bad, torch.full_like(s, float("nan")), s))
        s = torch.cat(scores)
        best = torch.sort(torch.nan_to_num(s, nan=-1.0), descending=True).values[:case["m"]]
        return dict(scores=s, valid=None, idx=None, best=best, count=None)
    if kind == "fit":
        X, y = _candidates(g, case)
        offs, D, m, k = _offsets(case), case["D"], case["m_sis"], case["k"]
        R, sub, sses = y[None], torch.empty(0, dtype=torch.int64, device=DEV), []
        for d in range(1, D + 1):
            s = torch.cat([_exact_scores(X[a:a + 16384], R, offs) for a in range(0, X.shape[0], 16384)])
            s = torch.nan_to_num(s, nan=-1.0)
            s[sub] = -1.0
            sub = torch.cat([sub, torch.argsort(s, descending=True, stable=True)[:m]])
            F = X[sub]
            sse, t = _exact_models(F, y, offs, d, k)
            sses.append(sse)
            R = []
            for q in t[:case["n_res"]]:
                r = torch.empty_like(y)
                for a, b in zip(offs[:-1], offs[1:]):
                    A = torch.cat([torch.ones(1, b - a, dtype=torch.float64, device=DEV), F[q, a:b]]).T
                    Q, _ = torch.linalg.qr(A)
                    r[a:b] = y[a:b] - Q @ (Q.T @ y[a:b])
                R.append(r)
            R = torch.stack(R)
        return dict(subspace=None, models=None, sse=torch.stack(sses), coef=None)
    if kind == "propose":
        return None  # the prefixes kept depend on the network's 16-bit scores
    st = prepare(case, seed)
    dt = torch.float64
    P, x, t = st["p"].to(dt), st["x"].to(dt), st["t"].to(dt)
    H, I = B.MLP_HIDDEN, B.MLP_IN
    parts = torch.split(P, [I * H, H, H * H, H, H, 1])
    w1, b1, w2, b2, w3, b3 = (q.clone().requires_grad_(True) for q in parts)
    h1 = torch.relu(x @ w1.reshape(I, H) + b1)
    h2 = torch.relu(h1 @ w2.reshape(H, H) + b2)
    out = h2 @ w3 + b3
    loss = (out - t).square().mean()
    loss.backward()
    grad = torch.cat([q.grad.reshape(-1) for q in (w1, b1, w2, b2, w3, b3)])
    m = 0.9 * st["m"].to(dt) + 0.1 * grad
    v = 0.999 * st["v"].to(dt) + 0.001 * grad * grad
    step = st["step"]
    p = P - case["lr"] * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
    return dict(out=out.detach(), grad=grad, loss=loss.detach()[None], params=p, m=m, v=v)
