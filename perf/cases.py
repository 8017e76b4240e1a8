"""The work that a Bayesian-optimisation loop has the library do, as timed cases.

One iteration of such a loop fits its models to the observations so far, scores a large
batch of candidate configurations, climbs from the best of them, and now and then fits
the hyperparameters again; spaces with known constraints also draw candidates from (and
test them against) a Chain-of-Trees, and a random forest may stand in for the classifier.
The search spaces are the five shapes that the repository's workloads and benchmark use:

  mixed     2 real, 1 integer, 1 log2 ordinal, 1 categorical (d = 5)
  schedule  loop-schedule space: ordinals, categorical, integers, a permutation (d = 6)
  tile      GPU-tile space: 10 log2 ordinals under known constraints
  pragma    FPGA-pragma space: 12 binary categoricals, 6 ordinals, 2 integers (d = 20)
  stress    6 ordinals, 2 real, 2 categoricals, 2 permutations, lengthscales from 0.1 to 10
"""
import math
import types

import numpy as np
import torch

from paper_2212_11142_amd import gp

DEV = "cuda"


# ------------------------------------------------------------------------------ spaces
def _param(kind, **kw):
    base = dict(kind=kind, log2=False, lo=0.0, hi=1.0, values=(), levels=0, m=0, dist="spearman")
    base.update(kw)
    return types.SimpleNamespace(**base)


def _pow2(count):
    return tuple(2 ** k for k in range(count))


def space_of(name):
    """(parameters, lengthscales) of a space."""
    if name == "mixed":
        ps = [_param("real"), _param("real"), _param("int", lo=1, hi=64),
              _param("ord", log2=True, values=_pow2(5)), _param("cat", levels=3)]
        return ps, np.full(5, 0.5)
    if name == "schedule":
        ps = [_param("ord", log2=True, values=_pow2(9)), _param("ord", log2=True, values=_pow2(4)),
              _param("cat", levels=3), _param("int", lo=1, hi=64), _param("int", lo=1, hi=32),
              _param("perm", m=5, dist="kendall")]
    elif name == "tile":
        ps = [_param("ord", log2=True, values=_pow2(11)) for _ in range(10)]
    elif name == "pragma":
        ps = ([_param("cat", levels=2) for _ in range(12)]
              + [_param("ord", log2=True, values=_pow2(6)) for _ in range(6)]
              + [_param("int", lo=1, hi=128) for _ in range(2)])
    else:
        ps = ([_param("ord", log2=True, values=_pow2(7)) for _ in range(6)]
              + [_param("real"), _param("real"), _param("cat", levels=8), _param("cat", levels=8),
                 _param("perm", m=7, dist="spearman"), _param("perm", m=7, dist="hamming")])
        return ps, np.exp(np.random.default_rng(1005).uniform(math.log(0.1), math.log(10.0), 12))
    return ps, np.full(len(ps), math.sqrt(len(ps)) / 2)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(shape, g):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)


def _ints(lo, hi, count, g):
    return torch.randint(lo, hi, (count,), generator=g, device=DEV, dtype=torch.int32)


def _uniform(ps, count, g):
    cols = []
    for p in ps:
        if p.kind == "real":
            cols.append(p.lo + (p.hi - p.lo) * _rand(count, g))
        elif p.kind == "int":
            cols.append(_ints(int(p.lo), int(p.hi) + 1, count, g))
        elif p.kind == "ord":
            cols.append(_ints(0, len(p.values), count, g))
        elif p.kind == "cat":
            cols.append(_ints(0, p.levels, count, g))
        else:
            cols.append(_rand((count, p.m), g).argsort(1).to(torch.int32).contiguous())
    return cols


def _tile_ok(c):
    """Known constraints of the tile space on level indices (G, L, T, vector width)."""
    ok = (c[3] + c[4] + c[5]) <= 10
    for k in range(3):
        ok &= (c[6 + k] <= c[3 + k]) & (c[3 + k] <= c[k])
    return ok & (c[9] <= c[6])


def _tile_draw(count, g):
    """Configurations inside the tile space's constraints."""
    u = _rand((10, count), g)
    a = (u[0] * 11).floor().clamp(max=10)
    b = (u[1] * (11 - a)).floor().minimum(10 - a)
    c = (u[2] * (11 - a - b)).floor().minimum(10 - a - b)
    L = [a, b, c]
    G = [L[k] + (u[3 + k] * (11 - L[k])).floor().minimum(10 - L[k]) for k in range(3)]
    T = [(u[6 + k] * (L[k] + 1)).floor().minimum(L[k]) for k in range(3)]
    V = (u[9] * (T[0] + 1)).floor().minimum(T[0])
    return [x.to(torch.int32).contiguous() for x in G + L + T + [V]]


def _tile_mixed(count, levels, g):
    """Half inside the constraints, half with one parameter set to another level."""
    cols = [c.clamp(max=levels - 1) for c in _tile_draw(count, g)]
    which, shift = _ints(0, 20, count, g), _ints(1, levels, count, g)
    return [torch.where(which == i, (c + shift) % levels, c).contiguous()
            for i, c in enumerate(cols)]


def _features(ps, cols):
    """Numeric features in [0, 1] for the synthetic objective."""
    fs = []
    for p, c in zip(ps, cols):
        x = c.double()
        if p.kind in ("real", "int"):
            fs.append((x - p.lo) / (p.hi - p.lo))
        elif p.kind == "ord":
            fs.append(x / (len(p.values) - 1))
        elif p.kind == "cat":
            fs.append(x / (p.levels - 1))
        else:
            fs.extend((x / (p.m - 1)).unbind(1))
    return torch.stack(fs, 1)


def _observe(name, ps, n, with_cls, g):
    """n observed configurations: columns, standardised log runtimes, feasibility flags."""
    X = _tile_draw(n, g) if name == "tile" else _uniform(ps, n, g)
    z = _features(ps, X)
    f = z.shape[1]
    nrm = lambda *s: torch.randn(s, generator=g, device=DEV, dtype=torch.float64)  # noqa: E731
    A = nrm(f, f) / math.sqrt(f)
    t = ((z @ A) ** 2).sum(1) / math.sqrt(f) + z @ nrm(f) + 0.1 * nrm(n)
    feas = torch.ones(n, dtype=torch.uint8, device=DEV)
    if with_cls:  # a hidden constraint: the top 30% of a noisy linear score fail
        feas[((z @ nrm(f)) + 0.1 * nrm(n)).argsort(descending=True)[:max(1, (3 * n) // 10)]] = 0
    ok = feas.bool()
    y = (t - t[ok].mean()) / t[ok].std()
    return X, torch.where(ok, y, torch.zeros_like(y)).contiguous(), feas


def _theta(d, count, seed):
    """Sampled hyperparameter settings: log lengthscales, log output scale, log noise."""
    lo = np.array([math.log(0.1)] * (d + 1) + [math.log(1e-6)])
    hi = np.array([math.log(10.0)] * (d + 1) + [0.0])
    return torch.from_numpy(lo + (hi - lo) * np.random.default_rng(seed).random((count, d + 2))).to(DEV)


_LEAVES = {}


def _tile_leaves(levels):
    """Every configuration of the tile space with so many levels inside the constraints, as
    level indices in lexicographic order: the table that a program with this space holds."""
    if levels not in _LEAVES:
        P = torch.zeros((1, 0), dtype=torch.int32, device=DEV)

        def grow(P, hi):
            cnt = (hi + 1).clamp(min=0).long()
            rows = torch.repeat_interleave(torch.arange(len(P), device=DEV), cnt)
            val = torch.arange(len(rows), device=DEV) - (cnt.cumsum(0) - cnt)[rows]
            return torch.cat([P[rows], val[:, None].to(torch.int32)], 1)

        for _ in range(3):
            P = grow(P, torch.full((len(P),), levels - 1, device=DEV))
        for k in range(3):
            P = grow(P, torch.minimum(P[:, k], 10 - P[:, 3:3 + k].sum(1, dtype=torch.int32)))
        for k in range(3):
            P = grow(P, P[:, 3 + k])
        _LEAVES.clear()
        _LEAVES[levels] = grow(P, P[:, 6])
    return _LEAVES[levels]


# ------------------------------------------------------------------------------- cases
def listed():
    return [
        # a kept model scores a small batch again and again: launches and latency
        {"name": "score_mixed", "kind": "score", "space": "mixed", "n": 32, "M": 4096, "cls": False},
        # one iteration at the evaluation budgets of a short tuning run
        {"name": "step_budget", "kind": "step", "space": "mixed", "n": 60, "M": 10007, "cls": True},
        # one iteration on a loop-schedule space, no hidden constraint
        {"name": "step_schedule", "kind": "step", "space": "schedule", "n": 128, "M": 65536, "cls": False},
        # a dense, masked batch near the data, with a hidden constraint
        {"name": "step_tile", "kind": "step", "space": "tile", "n": 256, "M": 262144, "cls": True},
        # the headline size of the benchmark
        {"name": "step_pragma", "kind": "step", "space": "pragma", "n": 512, "M": 1048576, "cls": True},
        # the largest: a long history and every parameter type
        {"name": "step_stress", "kind": "step", "space": "stress", "n": 2048, "M": 1048576, "cls": False},
        # a program that fits and scores in two calls, allocating as it goes, at odd sizes
        {"name": "fit_score_ragged", "kind": "fit_score", "space": "pragma", "n": 389, "M": 100003, "cls": True},
        # the acquisition optimiser's climb from the best of a scored batch
        {"name": "search_pragma", "kind": "search", "space": "pragma", "n": 512, "M": 262144, "cls": True, "starts": 8, "steps": 48},
        # the hyperparameter fit that a loop repeats as observations come in
        {"name": "hyperfit_schedule", "kind": "hyperfit", "space": "schedule", "n": 120, "samples": 128, "keep": 6, "iters": 12},
        # a batch of sampled settings with gradients, for a caller's own optimiser
        {"name": "posterior_pragma", "kind": "posterior", "space": "pragma", "n": 359, "count": 64},
        # the paper's own feasibility model: grown on the labels, applied to a batch
        {"name": "forest_pragma", "kind": "forest", "space": "pragma", "n": 512, "M": 1048576, "trees": 64},
        # known constraints: a uniform draw from the feasible set, and a mask of a batch
        {"name": "chain_tile", "kind": "chain", "space": "tile", "levels": 11, "M": 1048576},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["score", "step", "step", "step", "fit_score", "search", "hyperfit",
                       "posterior", "forest", "chain"])
    if kind == "chain":
        return {"kind": kind, "space": "tile", "levels": rng.randint(7, 11), "M": log_int(5000, 1048576)}
    space = rng.choice(["mixed", "schedule", "tile", "pragma", "stress"])
    cls = rng.random() < 0.5
    case = {"kind": kind, "space": space}
    if kind == "hyperfit":
        case.update(space=rng.choice(["mixed", "schedule", "pragma"]), n=log_int(24, 300),
                    samples=rng.randint(32, 256), keep=rng.randint(2, 8), iters=rng.randint(6, 12))
    elif kind == "posterior":
        case.update(n=log_int(24, 512), count=log_int(4, 128))
    elif kind == "forest":
        case.update(n=log_int(40, 1024), M=log_int(5000, 1048576), trees=log_int(16, 128))
    elif kind == "search":
        case.update(space=rng.choice(["schedule", "pragma", "stress"]), n=log_int(48, 700),
                    M=log_int(5000, 524288), cls=cls, starts=rng.randint(1, 12), steps=rng.randint(16, 48))
    else:
        # in the spaces of few dimensions a long history lies near every candidate, and most
        # are scored again in 64 bits: there a history of several hundred is already a long one
        most = 700 if space in ("mixed", "schedule", "tile") else 900 if cls else 2048
        case.update(n=log_int(24, most), M=log_int(1000, 1048576), cls=cls)
    return case


# ----------------------------------------------------------------------------- inputs
SIGNAL, NOISE, CLS_SIGNAL, FLOOR, PRIOR = 1.0, 1e-4, 1.0, 1e-6, (1.5, 1.0)


def _inputs(case, seed):
    """What both the library's call and the 64-bit reference take."""
    ps, ls = space_of(case["space"])
    g = _gen(seed)
    s = types.SimpleNamespace(case=case, ps=ps, ls=ls, mask=None)
    if case["kind"] == "chain":
        s.C = _tile_mixed(case["M"], case["levels"], g)
        s.seed = int(seed)
        return s
    s.X, s.y, s.feas = _observe(case["space"], ps, case["n"],
                                case.get("cls", False) or case["kind"] == "forest", g)
    s.cls = CLS_SIGNAL if case.get("cls", False) else None
    if "M" in case:
        s.C = _tile_mixed(case["M"], 11, g) if case["space"] == "tile" else _uniform(ps, case["M"], g)
        if case["space"] == "tile":
            s.mask = _tile_ok(s.C).to(torch.uint8)
    if case["kind"] == "forest":
        s.ei = _rand(case["M"], g).float()
        s.seed = int(seed) % 1000003
    if case["kind"] in ("hyperfit", "posterior"):
        s.theta = _theta(len(ps), case.get("samples", case.get("count")), seed)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    if kind == "chain":
        ps = [_param("ord", log2=True, values=_pow2(case["levels"])) for _ in range(10)]
        s.chain = gp.Chain(gp.Space(ps), [list(range(10))], [_tile_leaves(case["levels"])])
        return s
    s.space = gp.Space(s.ps)
    if kind in ("score", "search"):
        s.model = gp.fit(s.space, s.X, s.y, s.feas, s.ls, SIGNAL, NOISE, s.cls)
    if kind == "score":
        s.bufs = gp.ScoreBuffers(s.model, case["M"], want_argmax=True)
    if kind == "step":
        s.bufs = gp.FitScoreBuffers(s.space, case["n"], case["M"], with_cls=case["cls"], want_argmax=True)
    return s


def run(s):
    kind, case = s.case["kind"], s.case
    if kind == "score":
        gp.score_into(s.model, s.C, s.bufs, s.mask, 0.0)
        return s.bufs.result()
    if kind == "step":
        s.model = gp.fit_score_into(s.space, s.X, s.y, s.feas, s.ls, SIGNAL, NOISE, s.cls, s.C, s.bufs,
                                    s.mask, 0.0)
        return s.bufs.result()
    if kind == "fit_score":
        model = gp.fit(s.space, s.X, s.y, s.feas, s.ls, SIGNAL, NOISE, s.cls)
        out = gp.score(model, s.C, s.mask, 0.0, want_argmax=True)
        s.model = model  # the program goes on with it
        return {k: v for k, v in out.items() if k != "_buffers"}
    if kind == "search":
        return gp.local_search(s.model, s.C, s.mask, 0.0, n_starts=case["starts"], max_steps=case["steps"])
    if kind == "hyperfit":
        out = gp.hyperfit(s.space, s.X, s.y, s.feas, s.theta, case["keep"], PRIOR, FLOOR, max_iter=case["iters"])
        return {k: out[k] for k in ("theta", "value", "value0", "keep")}
    if kind == "posterior":
        return gp.log_posterior(s.space, s.X, s.y, s.feas, s.theta, PRIOR, FLOOR)
    if kind == "forest":
        forest = gp.Forest(s.space, s.X, s.feas, n_trees=case["trees"], max_depth=16, seed=s.seed)
        p, acq = forest.predict(s.C, s.ei, s.mask, 0.0)
        s.forest = forest
        return {"p": p, "acq": acq}
    return {"sample": s.chain.sample(case["M"], s.seed), "member": s.chain.member(s.C)}


def work(case):
    kind = case["kind"]
    if kind == "chain":
        # ten int32 columns written, ten read, a key read for each draw, a mask byte written
        return {"bytes": case["M"] * (40 + 8 + 40 + 1), "flops": 0}
    ps, _ = space_of(case["space"])
    d = len(ps)
    row = sum(8 if p.kind == "real" else 4 * p.m if p.kind == "perm" else 4 for p in ps)
    n = case["n"]
    nf = n - max(1, (3 * n) // 10) if case.get("cls") else n
    if kind in ("hyperfit", "posterior"):
        # per setting: kernel values, factorisation, inverse and its product, gradient sums
        grad = n * n * (2.0 * n / 3 + 2 * d)
        each = n * n * (n / 3.0 + d + 10)
        if kind == "posterior":
            return {"bytes": n * (row + 8) + case["count"] * (d + 2) * 16, "flops": case["count"] * (each + grad)}
        runs = case["samples"] * each + case["keep"] * (case["iters"] + 1) * (each + grad)
        return {"bytes": n * (row + 8) + case["samples"] * (d + 3) * 8, "flops": runs}
    M = case["M"]
    if kind == "forest":
        # a walk of about log2 n levels for each candidate and tree; the trees' sorts
        depth = math.log2(n)
        return {"bytes": M * (row + 4 + 4 + 4), "flops": case["trees"] * (2.0 * M * depth + 4 * n * depth * depth)}
    fit = nf ** 3 / 3.0 + nf ** 3 / 3.0 + n * n * (d + 10)
    if case["cls"]:
        fit += 6 * n ** 3 / 3.0 + n ** 3 / 3.0
    each = n * (3 * d + 10) + nf * (nf + 1) + 4 * nf + (n * (n + 1) + 4 * n if case["cls"] else 0)
    if kind == "search":
        # the batch scored for its starts, then every neighbour of every start at each move
        nb = sum(p.levels - 1 if p.kind == "cat" else p.m * (p.m - 1) // 2 if p.kind == "perm" else 2 for p in ps)
        rows = case["starts"] * nb * case["steps"] / 2
        return {"bytes": M * row + case["starts"] * row, "flops": M * n * (3 * d + 10) + rows * each}
    out = 4 * 5 + (1 if case["space"] == "tile" else 0)
    return {"bytes": M * (row + out) + n * (row + 9), "flops": M * each + (0 if kind == "score" else fit)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("forest", "chain"):
        return "exact"  # integer work, and one fixed-order mean in 64 bits
    if kind == "posterior":
        return {"rel": 1e-9}  # measured 2e-11 against the reference at small noise
    if kind == "hyperfit":
        return {"rel": 1e-6}  # measured 1e-10 where y differs by 1e-13 and iterations follow
    return {"rel": 2e-5}      # measured 5e-6 against the reference (scores in 32 bits)


# --------------------------------------------------------------------------- reference
def _codes(p, col):
    """The normalised numeric value of a parameter (in 64 bits, from its 32-bit code)."""
    if p.kind == "ord":
        t = np.array(p.values, dtype=np.float64)
        t = np.log2(t) if p.log2 else t
        v, lo, hi = torch.from_numpy(t).to(DEV)[col.long()], t[0], t[-1]
    else:
        v, lo, hi = col.double(), float(p.lo), float(p.hi)
    return ((v - lo) / (hi - lo)).float().double()


def _terms(ps, A, B):
    """Per parameter, the squared distance over its maximum between all rows of A and B."""
    for p, a, b in zip(ps, A, B):
        if p.kind == "cat":
            yield (a[:, None] != b[None, :]).double()
        elif p.kind != "perm":
            yield (_codes(p, a)[:, None] - _codes(p, b)[None, :]) ** 2
        elif p.dist == "spearman":
            yield ((a[:, None].double() - b[None, :].double()) ** 2).sum(2) / ((p.m ** 3 - p.m) / 3)
        elif p.dist == "hamming":
            yield (a[:, None] != b[None, :]).double().sum(2) / p.m
        else:
            i, j = torch.triu_indices(p.m, p.m, 1, device=DEV)
            oa, ob = a[:, i] > a[:, j], b[:, i] > b[:, j]
            yield (oa[:, None] != ob[None, :]).double().sum(2) / len(i)


def _matern(r2, sv):
    r = torch.sqrt(r2)
    return sv * (1.0 + math.sqrt(5.0) * r + 5.0 / 3.0 * r2) * torch.exp(-math.sqrt(5.0) * r)


def _kernel(ps, ls, A, B, sv):
    r2 = None
    for t, l in zip(_terms(ps, A, B), ls):
        r2 = t / l ** 2 if r2 is None else r2 + t / l ** 2
    return _matern(r2, sv)


def _phi(z):
    return torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)


def _cdf(z):
    return 0.5 * torch.erfc(-z / math.sqrt(2.0))


def _laplace(K, t):
    """Mode of the probit Laplace approximation: gradient, sqrt(W), chol(I + W^.5 K W^.5)."""
    f = torch.zeros_like(t)
    eye = torch.eye(len(t), dtype=torch.float64, device=DEV)
    for _ in range(100):
        z = t * f
        ratio = torch.exp(-0.5 * z * z - torch.special.log_ndtr(z)) / math.sqrt(2 * math.pi)
        g, W = t * ratio, ratio * (ratio + z)
        sw = torch.sqrt(W)
        L = torch.linalg.cholesky(eye + sw[:, None] * K * sw[None, :])
        b = W * f + g
        a = b - sw * torch.cholesky_solve((sw * (K @ b))[:, None], L)[:, 0]
        new = K @ a
        if float((new - f).abs().max()) < 1e-11:
            return g, sw, L
        f = new
    return g, sw, L


def _exact_score(s):
    ok = s.feas.bool()
    Xf = [c[ok] for c in s.X]
    K = _kernel(s.ps, s.ls, Xf, Xf, SIGNAL)
    nf = len(K)
    L = torch.linalg.cholesky(K + NOISE * torch.eye(nf, dtype=torch.float64, device=DEV))
    yf = s.y[ok]
    alpha = torch.cholesky_solve(yf[:, None], L)[:, 0]
    fstar = yf.min()
    inv = lambda T: torch.linalg.solve_triangular(  # noqa: E731
        T, torch.eye(len(T), dtype=torch.float64, device=DEV), upper=False)
    Lt = inv(L).T.contiguous()
    if s.cls is not None:
        grad, sw, LB = _laplace(_kernel(s.ps, s.ls, s.X, s.X, s.cls), torch.where(ok, 1.0, -1.0).double())
        LBt = inv(LB).T.contiguous()
    out = {k: [] for k in ("mu", "sigma", "ei", "acq", "p_feas")}
    M, step = s.case["M"], max(1024, int(4e7) // s.case["n"])
    for i in range(0, M, step):
        Ci = [c[i:i + step] for c in s.C]
        ks = _kernel(s.ps, s.ls, Ci, s.X, SIGNAL)
        kf = ks[:, ok]
        mu = kf @ alpha
        sg = torch.sqrt((SIGNAL - ((kf @ Lt) ** 2).sum(1)).clamp(min=0.0))
        z = (fstar - mu) / sg
        ei = ((fstar - mu) * _cdf(z) + sg * _phi(z)).clamp(min=0.0)
        p = torch.ones_like(mu)
        if s.cls is not None:
            kc = ks * (s.cls / SIGNAL)
            V = (s.cls - (((kc * sw[None, :]) @ LBt) ** 2).sum(1)).clamp(min=0.0)
            p = _cdf((kc @ grad) / torch.sqrt(1.0 + V))
        acq = torch.where(p > 0.0, ei * p, torch.zeros_like(p))
        if s.mask is not None:
            acq = torch.where(s.mask[i:i + step].bool(), acq, torch.zeros_like(acq))
        for k, x in (("mu", mu), ("sigma", sg), ("ei", ei), ("acq", acq), ("p_feas", p)):
            out[k].append(x)
    out = {k: torch.cat(v) for k, v in out.items()}
    return {**out, "argmax": None}


def _exact_posterior(s, want_grad):
    T = torch.stack(list(_terms(s.ps, s.X, s.X)))
    n, d = T.shape[1], T.shape[0]
    eye = torch.eye(n, dtype=torch.float64, device=DEV)
    off = 1.0 - eye
    vals, grads = [], []
    for th in s.theta:
        th = th.clone().requires_grad_(want_grad)
        r2 = torch.tensordot(torch.exp(-2.0 * th[:d]), T, dims=1)
        # off the diagonal only: a coincident pair's root has no derivative in autograd
        K = torch.where(r2 > 0, _matern(torch.where(r2 > 0, r2, off * 0 + 1.0), torch.exp(th[d])),
                        torch.exp(th[d]))
        L = torch.linalg.cholesky(K + (FLOOR + torch.exp(th[d + 1])) * eye)
        z = torch.linalg.solve_triangular(L, s.y[:, None], upper=False)
        a, b = PRIOR
        v = (-0.5 * (z * z).sum() - torch.log(torch.diagonal(L)).sum() - 0.5 * n * math.log(2 * math.pi)
             + (a * math.log(b) - math.lgamma(a) + (a - 1) * th[:d] - b * torch.exp(th[:d])).sum())
        if want_grad:
            grads.append(torch.autograd.grad(v, th)[0])
        vals.append(v.detach())
    return torch.stack(vals), (torch.stack(grads) if want_grad else None)


def exact(case, seed):
    if case["kind"] in ("chain", "forest", "search"):
        return None  # whole values, or trees and climbs that follow the library's own rules
    s = _inputs(case, seed)
    if case["kind"] == "posterior":
        value, grad = _exact_posterior(s, True)
        return {"value": value, "grad": grad}
    if case["kind"] == "hyperfit":
        return {"theta": None, "value": None, "value0": _exact_posterior(s, False)[0], "keep": None}
    return _exact_score(s)
