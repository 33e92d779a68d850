"""The 16-lane top-k of scored rows against the oracle at the edges of its
register blocks (1 to 891 candidates per row), k from 1 to 16, with rows of
exact ties (features 0 or 1, integer offsets: the id order must match) and rows
with fewer valid candidates than k."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_16849_amd import snls as B
from tests.parity import compare_topk
from workloads import small_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ws,wt,T,k,ties,dist", [
    (1, 0, 2, 1, False, 0), (8, 0, 1, 16, False, 0), (9, 0, 2, 13, True, 0), (5, 2, 3, 10, False, 1),
    (9, 1, 2, 16, True, 1), (9, 2, 5, 10, False, 0), (9, 2, 1, 16, True, 0), (9, 3, 4, 14, False, 0),
    (9, 5, 3, 12, True, 0), (3, 2, 1, 16, False, 1),
])
def test_group_topk(ws, wt, T, k, ties, dist):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    p = small_params(T=T, C=8, H=13, W=14, ws=ws, wt=wt, ps=3, k=k, dist_type=dist)
    rng = np.random.default_rng(ws * 100 + k)
    shp, fshp = (1, T, 8, 13, 14), (1, T, 2 * wt, 2, 13, 14)
    if ties:
        q, kk = (rng.integers(0, 2, shp).astype(np.float32) for _ in range(2))
        fl = rng.integers(-3, 4, fshp).astype(np.float32)
    else:
        q, kk = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
        fl = rng.uniform(-9, 9, fshp).astype(np.float32)
    to = lambda a: torch.from_numpy(a).to(dev)
    gd, gi = B.snls_search(to(q), to(kk), to(fl) if wt else None, p)
    torch.cuda.synchronize()
    gd, gi = gd.cpu().numpy().reshape(-1, k), gi.cpu().numpy().reshape(-1, k, 3)
    res = oracle.search(q, kk, fl, p)
    n, _ = compare_topk(gd, gi, res, k)
    if ties:
        assert n == 0 and np.array_equal(gd, res["dists"][:, :k].astype(np.float32))


@pytest.mark.parametrize("ps,C", [(1, 8), (3, 16), (7, 4)])
@pytest.mark.parametrize("what", [np.nan, np.inf])
def test_every_candidate_kept_with_features_that_are_not_finite(ps, C, what):
    """NaN and infinite features up to the frame's borders: the scores of a
    search that keeps every candidate are those of the direct sums, invalid
    only where a pixel of the patch inside the frame gives NaN.  The keys' ones
    are in frame 1 and the queries compared in frame 0, half offsets away (no
    tap has weight 0)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    p = small_params(T=2, C=C, H=22, W=25, ws=5, wt=1, ps=ps, k=0)
    rng = np.random.default_rng(C)
    shp = (1, 2, C, 22, 25)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    for a, f in ((q, 0), (k, 1)):
        for _ in range(6):
            a[0, f, rng.integers(0, C), rng.integers(0, 22), rng.integers(0, 25)] = what * rng.choice([1, -1])
        a[0, f, 3, 0, 5] = a[0, f, 2, 21, 24] = a[0, f, 1, 12, 0] = what
    fl = (rng.integers(-3, 3, (1, 2, 2, 2, 22, 25)) + 0.5).astype(np.float32)
    d = lambda a: torch.from_numpy(a).to(dev)
    gd, _ = B.snls_search(d(q), d(k), d(fl), p)
    n = 22 * 25
    gd, ref = gd.cpu().numpy().reshape(-1, 75)[:n], oracle.search(q, k, fl, dict(p, k=4))["all_dists"][:n]
    fin = np.isfinite(ref)
    assert not np.isnan(gd).any() and np.array_equal(gd[~fin], ref[~fin])
    assert np.abs(gd[fin] - ref[fin]).max() <= 1e-5 * ps * ps * np.sqrt(C)
