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
