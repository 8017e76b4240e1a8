"""GPU tests at the sizes where a kernel's tiles, remainders or dispatch rules change."""
import numpy as np
import pytest

from workloads import make_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _announce(request):
    print(f"\n[gpu] {request.node.nodeid}", flush=True)
    yield


def _fit(w, n=None, noise=None):
    import torch

    from paper_2212_11142_amd import gp
    space = gp.Space(w.space)
    X = gp.to_device_columns(space, w.X)
    y = torch.from_numpy(np.nan_to_num(w.y, nan=0.0)).cuda()
    feas = torch.from_numpy(w.feasible).cuda()
    return space, gp.fit(space, X, y, feas, w.lengthscale, w.signal_var,
                         w.noise_var if noise is None else noise, w.cls_signal_var)


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 15, 16, 17, 19, 20, 31, 32, 33, 47, 48, 49, 63, 64,
                               65, 97])
def test_block_factorisation_sizes(n):
    """L, L^-1 and alpha at every remainder class of the 32-wide blocks, their 16-wide tiles
    and 4-wide panels. Bounds: a backward-stable factorisation leaves n eps |K| in L L^T
    and n eps cond(L) in L^-1 L; ten times those."""
    w = make_workload("C1", 128, n=n)
    _, model = _fit(w)
    K, L, Li = model.export("K"), model.export("L"), model.export("LINV")
    eps = np.finfo(np.float64).eps
    assert np.abs(L @ L.T - K).max() <= 10 * n * eps * np.abs(K).max()
    assert np.all(np.triu(L, 1) == 0) and np.all(np.diag(L) > 0)
    assert np.abs(Li @ L - np.eye(n)).max() <= 10 * n * eps * np.linalg.cond(L)
    ref = np.linalg.solve(K, w.y)
    assert np.abs(model.export("ALPHA") - ref).max() <= 10 * n * eps * np.linalg.cond(K) * np.abs(ref).max()


@pytest.mark.parametrize("dup", [1, 3, 4, 15, 16, 17, 30, 31, 32, 40])
def test_block_factorisation_failing_pivot(dup):
    """Without noise a repeated observation makes its own pivot the first that fails (to
    rounding: it may come out as a tiny positive number, then the fit succeeds with a
    Gram matrix singular to working precision)."""
    from paper_2212_11142_amd import gp
    w = make_workload("C1", 128, n=48)
    for c in w.X:
        c[dup] = c[0]
    try:
        _, model = _fit(w, noise=0.0)
    except gp.GPError as e:
        assert e.status == 2 and f"pivot {dup} " in str(e)
    else:
        assert model.export("L")[dup, dup] <= 1e-6


@pytest.mark.parametrize("k", [1, 8, 63, 64])
@pytest.mark.parametrize("M", [1, 3, 64, 65, 1023, 1024, 1025, 2049, 5000, 65535])
def test_start_selection(M, k):
    """The starts of a search are the k largest values, lower index first on ties (a mask
    makes many equal zeros), at the edges of the selection's batches and block counts."""
    import torch

    from paper_2212_11142_amd import gp
    w = make_workload("C1", 65536, n=20)
    space, model = _fit(w)
    Cc = [c[:M].contiguous() for c in gp.to_device_columns(space, w.C)]
    mask = (torch.arange(M, device="cuda") % 3 == 1).to(torch.uint8)
    acq = gp.score(model, Cc, mask=mask)["acq"].cpu().numpy()
    out = gp.local_search(model, Cc, mask=mask, n_starts=k, max_steps=0)
    want = np.lexsort((np.arange(M), -acq))[:min(k, M)]
    assert np.array_equal(out["start_index"].cpu().numpy(), want)
    assert np.array_equal(out["acq"].cpu().numpy(), acq[want])


@pytest.mark.parametrize("k", [1, 64])
@pytest.mark.parametrize("M", [63, 127, 129, 16383, 16384, 16385])
def test_start_selection_blocks(M, k):
    """The same where the number of blocks and the elements of a block change."""
    test_start_selection(M, k)


@pytest.mark.parametrize("order", ["drawn", "ascending"])
@pytest.mark.parametrize("M", [262145, 600001])
def test_start_selection_many_batches(M, order):
    """Ranges of more than one batch per block: the threshold that a block keeps, and its
    sort before the range ends; ascending values pass every threshold."""
    import torch

    from paper_2212_11142_amd import gp
    w = make_workload("C1", M, n=20)
    space, model = _fit(w)
    Cc = gp.to_device_columns(space, w.C)
    if order == "ascending":
        by = torch.argsort(gp.score(model, Cc)["acq"], stable=True)
        Cc = [c[by].contiguous() for c in Cc]
    acq = gp.score(model, Cc)["acq"].cpu().numpy()
    want = np.lexsort((np.arange(M), -acq))
    for k in (1, 7, 64):
        out = gp.local_search(model, Cc, n_starts=k, max_steps=0)
        assert np.array_equal(out["start_index"].cpu().numpy(), want[:k])
        assert np.array_equal(out["acq"].cpu().numpy(), acq[want[:k]])


@pytest.mark.parametrize("sizes", [[1], [2], [4], [5], [6], [7], [39], [41], [300000],
                                   [1, 5, 5000, 200000]])
def test_chain_membership_tables(sizes):
    """Membership against numpy at the edges of its hash buckets: one bucket partly filled
    (wrapping onto itself), one key more than it holds on average, many buckets, several
    trees; first and last leaves, their neighbours and values out of range among the
    configurations."""
    import torch

    from paper_2212_11142_amd import gp
    from workloads import Param
    rng = np.random.default_rng(7)
    params = [Param(f"i{q}", "int", lo=-3, hi=1 << 19) for q in range(2 * len(sizes))]
    leaves, keep = [], []
    for s in sizes:
        rows = np.unique(rng.integers(0, 1 << 19, size=(2 * s + 8, 2)), axis=0)
        rows = rows[np.sort(rng.choice(len(rows), s, replace=False))].astype(np.int32)
        leaves.append(rows)
        keep.append(set(map(tuple, rows.tolist())))
    chain = gp.Chain(gp.Space(params), [[2 * t, 2 * t + 1] for t in range(len(sizes))], leaves)
    M = 4099
    cols, want = [], np.ones(M, bool)
    for t, rows in enumerate(leaves):
        pick = rows[rng.integers(0, len(rows), M)].astype(np.int64)
        pick[:2] = rows[[0, -1]]
        pick[2:4] = rows[[0, -1]] + [[0, -1], [0, 1]]
        off = rng.random(M) < 0.2
        pick[off, 1] += rng.integers(-2, 3, off.sum())
        pick[rng.random(M) < 0.02, 0] += 1 << 19
        want &= np.array([tuple(r) in keep[t] for r in pick.tolist()])
        cols += [pick[:, 0] - 3, pick[:, 1] - 3]   # raw values: lo + index
    got = chain.member([torch.from_numpy(c.astype(np.int32)).cuda() for c in cols]).cpu().numpy()
    assert np.array_equal(got.astype(bool), want)


def test_chain_membership_all_ones_key():
    """A key of 64 one bits (two 32-bit fields at their last value) is a member only if it is
    a leaf."""
    import torch

    from paper_2212_11142_amd import gp
    from workloads import Param
    params = [Param(f"c{q}", "cat", levels=65536) for q in range(4)]
    top = [65535] * 4
    for rows in ([[0, 1, 2, 3], top], [[0, 1, 2, 3], [65535, 65535, 65535, 65534]]):
        chain = gp.Chain(gp.Space(params), [[0, 1, 2, 3]], [np.array(rows, np.int32)])
        conf = np.array([top, [0, 1, 2, 3], [65535, 65535, 65535, 65534]], np.int32)
        cols = [torch.from_numpy(np.ascontiguousarray(conf[:, q])).cuda() for q in range(4)]
        want = [1 if c in rows else 0 for c in conf.tolist()]
        assert chain.member(cols).cpu().tolist() == want


@pytest.mark.parametrize("n,trees,depth,min_split", [
    (1, 3, 4, 2), (2, 5, 4, 1), (63, 4, 20, 2), (64, 4, 20, 2), (65, 4, 20, 2), (66, 7, 3, 9),
    (130, 3, 40, 2), (1025, 3, 40, 2), (2049, 2, 40, 2), (4096, 2, 40, 2)])
def test_forest_sizes(n, trees, depth, min_split):
    """Trees against the oracle, node for node, where the growth changes form: nodes of up to
    64 samples and above, ranks of many distinct values, wide levels, odd tree counts; and
    predictions against walking the returned trees (the same sum in the same order)."""
    import torch

    from oracle import gp_forest as of
    from paper_2212_11142_amd import gp
    w = make_workload("C1", 700, n=n)
    rng = np.random.default_rng(n)
    feas = (rng.random(n) < 0.6).astype(np.uint8)
    space = gp.Space(w.space)
    X = gp.to_device_columns(space, w.X)
    forest = gp.Forest(space, X, torch.from_numpy(feas).cuda(), n_trees=trees, max_depth=depth,
                  min_split=min_split, seed=11)
    ref = of.fit_forest(w.space, w.X, feas, trees, 11, depth, min_split)
    got = [forest.tree(t) for t in range(trees)]
    for t in range(trees):
        r = ref[t]
        val = [th if f >= 0 else v for f, th, v in zip(r.feature, r.threshold, r.value)]
        for a, b in zip(got[t], (r.feature, r.left, val)):
            assert np.array_equal(a, np.array(b))
    F = of.features(w.space, w.C)
    want = np.zeros(700)
    for feat, left, val in got:
        k = np.zeros(700, np.int64)
        while np.any(feat[k] >= 0):
            go = feat[k] >= 0
            x = F[np.arange(700), np.maximum(feat[k], 0)]
            k = np.where(go, left[k] + np.where(x <= val[k], 0, 1), k)
        want += val[k]
    p, _ = forest.predict(gp.to_device_columns(space, w.C))
    assert np.array_equal(p.cpu().numpy(), (want / trees).astype(np.float32))


@pytest.mark.parametrize("name,n,trees,M", [
    ("C5", 300, 1, 4099), ("C5", 300, 20, 4099), ("C5", 300, 40, 4099), ("C5", 300, 3, 131073),
    ("C5", 300, 4, 131073), ("C1", 200, 9, 4099), ("C1", 200, 12, 4099), ("C1", 200, 9, 131072),
    ("C1", 200, 9, 131073), ("C1", 200, 10, 131073), ("C1", 3071, 30, 1), ("C1", 3072, 30, 1),
    ("C1", 1024, 129, 5003), ("C1", 1024, 129, 262144 + 65)])
def test_forest_prediction_routes(name, n, trees, M):
    """Predictions on both sides of the rule between walks through the caches and through
    LDS, and by more trees than the LDS holds at once (several batches, read again for a
    workgroup's second set of configurations), against walking the returned trees: the same
    comparisons and the same sum in the same order. REAL values hold NaN (goes right),
    infinities, both zeros, values of the observations and values outside their range."""
    import torch

    from oracle import gp_forest as of
    from paper_2212_11142_amd import gp
    w = make_workload(name, M, n=n) if name == "C1" else make_workload(name, M)
    X = [c[:n] for c in w.X]
    C = [c.copy() for c in w.C]
    for q, p in enumerate(w.space):
        if p.kind == "real":
            odd = [np.nan, np.inf, -np.inf, 0.0, -0.0, -5.0, 5.0, X[q][0], X[q][n // 2]]
            C[q][:min(9, M)] = odd[:min(9, M)]
    rng = np.random.default_rng(M + trees)
    feas = (rng.random(n) < 0.6).astype(np.uint8)
    space = gp.Space(w.space)
    forest = gp.Forest(space, gp.to_device_columns(space, X), torch.from_numpy(feas).cuda(),
                       n_trees=trees, max_depth=40, seed=4)
    ei, mask = rng.random(M).astype(np.float32), (rng.random(M) < 0.8).astype(np.uint8)
    p, acq = forest.predict(gp.to_device_columns(space, C), torch.from_numpy(ei).cuda(),
                            torch.from_numpy(mask).cuda(), 0.3)
    p, acq = p.cpu().numpy(), acq.cpu().numpy()
    rows = np.unique(np.concatenate([np.arange(min(M, 16)), rng.integers(0, M, min(M, 4096)),
                                     np.arange(max(0, M - 130), M)]))
    F = of.features(w.space, [c[rows] for c in C])
    at, want, nodes = np.arange(len(rows)), np.zeros(len(rows)), 0
    for t in range(trees):
        feat, left, val = forest.tree(t)
        nodes += len(feat)
        k = np.zeros(len(rows), np.int64)
        while np.any(feat[k] >= 0):
            x = F[at, np.maximum(feat[k], 0)]
            k = np.where(feat[k] >= 0, left[k] + np.where(x <= val[k], 0, 1), k)
        want += val[k]
    assert trees < 100 or nodes > 160 * 1024 // 8  # more than one batch
    want = (want / trees).astype(np.float32)
    assert np.array_equal(p[rows], want)
    ok = (mask[rows] != 0) & (want > np.float32(0.3))
    assert np.array_equal(acq[rows], np.where(ok, ei[rows] * want, np.float32(0.0)))


@pytest.mark.parametrize("name", ["C3", "C4"])
def test_few_rows_bit_identical(name):
    """Batches small enough for the few-rows contraction and the one-block cross-kernel give
    the bits that the same candidates have inside a batch that takes the large tiles (every
    column tile, the classifier's dense column among them)."""
    import torch

    from paper_2212_11142_amd import gp
    w = make_workload(name, 16384)
    _, model = _fit(w)
    C = gp.to_device_columns(gp.Space(w.space), w.C)
    big = gp.score(model, C)
    for M in (1, 127, 128, 129, 300, 511, 640, 1025):
        small = gp.score(model, [c[:M].contiguous() for c in C])
        for k in ("sigma", "p_feas"):
            assert torch.equal(small[k], big[k][:M]), (k, M)


def test_one_block_cross_kernel_bit_identical():
    """The same for the cross-kernel with two candidate blocks per wavefront (permutations,
    n = 2048) on both sides of its one-block form's limit: 384 and 512 rows in 64 splits are
    768 and 1024 wavefronts. (mu is summed in as many parts as there are splits.)"""
    import torch

    from paper_2212_11142_amd import gp
    w = make_workload("C5", 4096)
    _, model = _fit(w)
    C = gp.to_device_columns(gp.Space(w.space), w.C)
    big = gp.score(model, C)
    for M in (1, 128, 129, 384, 385, 512, 513):
        small = gp.score(model, [c[:M].contiguous() for c in C])
        assert torch.equal(small["sigma"], big["sigma"][:M]), M
        assert float((small["mu"] - big["mu"][:M]).abs().max()) <= 4e-7 * float(big["mu"].abs().max())


@pytest.mark.parametrize("name,M", [("C4", 1024), ("C4", 1025), ("C4", 1536), ("C4", 1537),
                                    ("C3", 1536), ("C3", 1537), ("C3", 2048), ("C3", 2049)])
def test_few_rows_fused(name, M):
    """A fused step's value model has 3 (C4) or 2 (C3) column tiles on three quarters of the
    compute units: on both sides of the few-rows contraction's limits there (24 tiles, 36
    where k is long) and on the whole card (32, 48), it gives the bits of a separate fit and
    scoring."""
    import torch

    from paper_2212_11142_amd import gp
    w = make_workload(name, M)
    space, model = _fit(w)
    X, C = gp.to_device_columns(space, w.X), gp.to_device_columns(space, w.C)
    y = torch.from_numpy(np.nan_to_num(w.y, nan=0.0)).cuda()
    feas = torch.from_numpy(w.feasible).cuda()
    ref = gp.score(model, C)
    bufs = gp.FitScoreBuffers(space, len(w.y), M, with_cls=True)
    gp.fit_score_into(space, X, y, feas, w.lengthscale, w.signal_var, w.noise_var,
                      w.cls_signal_var, C, bufs)
    out = bufs.result()
    for k in ("mu", "sigma", "ei", "acq", "p_feas"):
        assert torch.equal(out[k], ref[k]), k


@pytest.mark.parametrize("d,n,count", [(1, 1, 1), (1, 2, 16), (7, 15, 17), (8, 16, 3), (9, 17, 33),
                                       (16, 33, 5), (17, 31, 15), (24, 65, 2), (25, 40, 64),
                                       (32, 50, 65), (33, 35, 4), (64, 48, 3)])
def test_log_posterior_shapes(d, n, count):
    """Objective and gradient at the edges of the matrix-product tiles: 16 settings, 16
    pairs, 4-wide steps and 16-wide tiles of parameters. Tolerances: fp64 sums of up to n^2
    terms behind a factorisation with noise 1e-2 or more (condition below 1e5)."""
    import torch

    from oracle import gp_hyper as gh
    from paper_2212_11142_amd import gp
    from workloads import Param
    rng = np.random.default_rng(d * 1000 + n)
    params = [Param(f"r{q}", "real") if q % 3 else Param(f"c{q}", "cat", levels=4) for q in range(d)]
    X = [rng.random(n) if p.kind == "real" else rng.integers(0, 4, n).astype(np.int32) for p in params]
    y, feas = rng.normal(size=n), np.ones(n, np.uint8)
    theta = rng.uniform(-1.0, 1.0, size=(count, d + 2))
    theta[:, d + 1] = rng.uniform(np.log(1e-2), 0.0, size=count)
    space = gp.Space(params)
    out = gp.log_posterior(space, gp.to_device_columns(space, X), torch.from_numpy(y).cuda(),
                           torch.from_numpy(feas).cuda(), torch.from_numpy(theta).cuda(), (1.5, 1.0))
    T, yf = gh.hyper_data(params, X, y, feas)
    for b in range(count):
        rv, rg = gh.log_posterior(T, yf, theta[b], (1.5, 1.0), 1e-6)
        assert abs(out["value"][b].item() - rv) <= 1e-10 * max(abs(rv), 1.0)
        assert np.abs(out["grad"][b].cpu().numpy() - rg).max() <= 1e-9 * max(np.abs(rg).max(), 1.0)


@pytest.mark.parametrize("n", [3, 31, 32, 63, 65, 200, 256, 257, 513, 1024, 1025])
def test_refine_block_sizes(n):
    """Every candidate recomputed in fp64 in groups (more than 4096 flagged) gives what the
    small-count path gives, at the edges of its observation chunks, column blocks and forms,
    with a ragged last group. Both are fp64 sums rounded to fp32 (mu, sigma, EI); the sum of
    squares is 1 - sigma^2, so sigma's bound grows as it cancels: n eps / sigma^2 with the
    fp32 rounding on top."""
    import torch

    from paper_2212_11142_amd import gp
    M = 4096 + 33
    w = make_workload("C1", M, n=n)
    space, model = _fit(w)
    gp.debug_set_refine(model, float("inf"), -1.0)
    C = gp.to_device_columns(space, w.C)
    big = gp.score(model, C)
    parts = [gp.score(model, [c[a:a + 100].contiguous() for c in C]) for a in (0, 2000, M - 100)]
    for a, p in zip((0, 2000, M - 100), parts):
        for k in ("mu", "sigma", "ei"):
            x, y = big[k][a:a + 100].double(), p[k].double()
            tol = 4e-7 * torch.maximum(y.abs(), torch.full_like(y, 1e-3 if k == "mu" else 0.0))
            if k != "mu":  # eps n cond of the cancellation, in units of sigma
                tol = tol + 1e-14 * n / p["sigma"].double().clamp(min=1e-3)
            assert bool(((x - y).abs() <= tol).all()), (k, a, float((x - y).abs().max()))


@pytest.mark.parametrize("n_real,n", [(40, 65), (30, 200), (30, 256), (16, 389), (16, 512), (24, 300),
                                      (40, 1000)])
def test_refine_block_streamed(n_real, n):
    """The same where the observations' codes do not stay in LDS: a chunk's are loaded between
    the phases, the next group's candidates beside them (not with the most column blocks).
    Noise 1e-2 keeps sigma^2 above 1e-3 of the signal variance: the sum of squares cancels
    n eps / 1e-3 at most, below the fp32 rounding of the outputs (6e-8, for mu of its sum's
    terms)."""
    import torch

    from paper_2212_11142_amd import gp
    from workloads import Param
    params = ([Param(f"r{q}", "real") for q in range(n_real)]
              + [Param("c", "cat", levels=5), Param("p", "perm", m=5)])
    ni, obs = 2, (n + 63) // 64 * 64  # words of the codes besides the numeric ones, at least
    lds = 8 * (32 * 66 + 24 * 32 + n_real * (64 + obs)) + 4 * ni * (64 + obs)
    assert lds > 78 * 1024  # (not resident)
    rng = np.random.default_rng(n)
    M = 4096 + 33

    def draw(count):
        cols = [rng.random(count) for _ in range(n_real)]
        cols.append(rng.integers(0, 5, count).astype(np.int32))
        cols.append(np.argsort(rng.random((count, 5)), axis=1).astype(np.int32))
        return cols

    space = gp.Space(params)
    X, C = gp.to_device_columns(space, draw(n)), gp.to_device_columns(space, draw(M))
    y = torch.from_numpy(rng.normal(size=n)).cuda()
    feas = torch.ones(n, dtype=torch.uint8, device="cuda")
    model = gp.fit(space, X, y, feas, np.full(n_real + 2, np.sqrt(n_real + 2) / 2), 1.0, 1e-2, None)
    gp.debug_set_refine(model, float("inf"), -1.0)
    big = gp.score(model, C)
    assert float(big["sigma"].min()) ** 2 > 1e-3
    assert gp.refined_count(model, big["_buffers"]) == M
    scale = float(big["mu"].abs().max())
    for a in (0, 2000, M - 100):
        p = gp.score(model, [c[a:a + 100].contiguous() for c in C])
        for k in ("mu", "sigma", "ei"):
            x, r = big[k][a:a + 100].double(), p[k].double()
            tol = 4e-7 * (torch.full_like(r, scale) if k == "mu" else r.abs() + 1e-7)
            assert bool(((x - r).abs() <= tol).all()), (k, a, float((x - r).abs().max()))


@pytest.mark.parametrize("M", [1, 2, 63, 64, 65, 1023, 1025, 32767, 32768, 32769])
def test_argmax_sizes(M):
    """The arg-max (lowest index on ties) on both sides of its one-workgroup form: free, and
    with all but a few masked off, where most values tie at zero."""
    import torch

    from paper_2212_11142_amd import gp
    w = make_workload("C1", 36864, n=20)
    space, model = _fit(w)
    C = [c[:M].contiguous() for c in gp.to_device_columns(space, w.C)]
    for mask in (None, torch.zeros(M, dtype=torch.uint8, device="cuda"),
                 (torch.arange(M, device="cuda") % 997 == 996).to(torch.uint8)):
        out = gp.score(model, C, mask=mask, want_argmax=True)
        assert int(out["argmax"][0]) == int(np.argmax(out["acq"].cpu().numpy()))
