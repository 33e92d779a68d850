"""The matrix-core scores of the tiled search against the oracle where the
kernel changes path: channel padding and chunk groups (8 to 130 channels per
head), unions of shift columns at the edges of two and three key blocks and of
the three lane layouts (17/18, 21/22, 32/33 columns) and of several sweeps, more
shift rows than one round holds, strided queries, every patch size, pixels and
channels of very different size, and values that are not finite."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_16849_amd import snls as B
from tests.parity import compare_topk
from workloads import small_params

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.load_library()
    return torch.device("cuda:0")


def _flows(p, rows, cols, rng):
    """Offsets whose integer parts spread over `rows` x `cols` shifts in every tile."""
    shp = (p["B"], p["T"], 2 * p["wt"], p["H"], p["W"])
    y, x = np.mgrid[0:p["H"], 0:p["W"]]
    fl = np.empty(shp[:3] + (2,) + shp[3:], np.float32)
    fl[:, :, :, 0] = 0.3 - rows // 2 + (y * 5 + x) % (rows + 1)
    fl[:, :, :, 1] = 0.6 - cols // 2 + (y + x * 3) % (cols + 1)
    return (fl + rng.uniform(-0.2, 0.2, fl.shape)).astype(np.float32)


def _search(q, k, fl, p, dev):
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    gd, gi = B.snls_search(d(q), d(k), d(fl), p)
    torch.cuda.synchronize()
    return gd.cpu().numpy().reshape(-1, p["k"]), gi.cpu().numpy().reshape(-1, p["k"], 3)


CASES = [  # patch, channels, heads, window, query stride, key stride, spread of rows and columns
    (7, 8, 1, 9, 1, 1.0, 4, 7), (7, 64, 1, 9, 1, 1.0, 6, 8), (7, 65, 1, 9, 1, 1.0, 14, 11), (3, 33, 1, 9, 1, 1.0, 7, 12),
    (5, 130, 1, 5, 1, 0.5, 3, 18), (7, 96, 3, 9, 1, 1.0, 26, 22), (1, 32, 1, 9, 1, 0.5, 5, 27), (2, 24, 2, 7, 1, 1.0, 9, 24),
    (4, 16, 1, 8, 2, 1.0, 8, 11), (6, 40, 1, 9, 3, 0.75, 5, 6), (7, 16, 1, 15, 1, 1.0, 3, 3), (7, 72, 1, 13, 2, 1.0, 9, 19), (7, 15, 1, 9, 2, 1.0, 5, 6),
    (7, 16, 1, 9, 2, 1.0, 5, 6),
]


@pytest.mark.parametrize("ps,C,HD,ws,s0,s1,rows,cols", CASES)
def test_scores_at_path_edges(dev, ps, C, HD, ws, s0, s1, rows, cols):
    p = small_params(T=2, C=C, HD=HD, H=38, W=43, ws=ws, wt=1, ps=ps, k=12, stride0=s0, stride1=s1)
    rng = np.random.default_rng(ps * 1000 + C)
    shp = (1, 2, C, 38, 43)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    fl = _flows(p, rows, cols, rng)
    gd, gi = _search(q, k, fl, p, dev)
    compare_topk(gd, gi, oracle.search(q, k, fl, p), p["k"])


@pytest.mark.parametrize("ps,C,s0,s1,cols,dark", [(7, 64, 1, 1.0, 55, False), (7, 72, 2, 0.5, 56, False), (3, 33, 1, 1.0, 88, True),
                                                  (5, 16, 3, 1.0, 60, False), (1, 32, 1, 1.0, 23, False), (1, 32, 1, 1.0, 70, False)])
def test_unions_swept_by_columns(dev, ps, C, s0, s1, cols, dark):
    """Unions of shift columns around one, two, three and four sweeps of 32
    (windows of 9 add 9 columns, at half strides 5), also with scales per pixel."""
    p = small_params(T=2, C=C, H=40, W=120, ws=9, wt=1, ps=ps, k=12, stride0=s0, stride1=s1)
    rng = np.random.default_rng(ps + cols)
    shp = (1, 2, C, 40, 120)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    if dark:
        q[..., ::7, ::5] *= 1e-6
    fl = rng.uniform(-2, 2, (1, 2, 2, 2, 40, 120)).astype(np.float32)
    x = np.arange(120) % 20 >= 10
    fl[:, :, :, 1] += np.where(x, cols - cols // 2, -(cols // 2)) - 0.5
    gd, gi = _search(q, k, fl, p, dev)
    compare_topk(gd, gi, oracle.search(q, k, fl, p), p["k"])


@pytest.mark.parametrize("ps,C,ws,s0,s1,cols,dist", [(7, 256, 9, 1, 1.0, 5, 0), (7, 193, 3, 1, 1.0, 14, 0), (5, 384, 9, 2, 0.5, 20, 0),
                                                     (3, 512, 5, 1, 1.0, 31, 0), (6, 320, 7, 3, 1.0, 50, 0), (7, 200, 9, 1, 1.0, 8, 1),
                                                     (1, 160, 9, 1, 1.0, 16, 0)])
def test_heads_of_many_channels(dev, ps, C, ws, s0, s1, cols, dist):
    """Three channel groups and more: the window tables collect the groups'
    sums (lane layouts of two and three parts, one and several sweeps)."""
    p = small_params(T=2, C=C, H=33, W=75, ws=ws, wt=1, ps=ps, k=12, stride0=s0, stride1=s1, dist_type=dist)
    rng = np.random.default_rng(ps * C)
    shp = (1, 2, C, 33, 75)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    fl = _flows(p, 5, cols, rng)
    gd, gi = _search(q, k, fl, p, dev)
    compare_topk(gd, gi, oracle.search(q, k, fl, p), p["k"])


@pytest.mark.parametrize("H,s0", [(18100, 1), (18100, 8)])
def test_tall_frames(dev, H, s0):
    """Valid offsets of one tile more than 16384 rows apart: a query's shift
    rows, relative to the tile's, leave 16 bits."""
    p = small_params(T=2, C=16, H=H, W=6, ws=3, wt=1, ps=3, k=9, stride0=s0)
    rng = np.random.default_rng(H + s0)
    shp = (1, 2, 16, H, 6)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    fl = rng.uniform(-1, 1, (1, 2, 2, 2, H, 6)).astype(np.float32)
    for i in range(0, 120, 24):  # from near the bottom to the top, and back
        top, bottom = 8 + i, (H - 128) // 8 * 8 + i
        fl[:, :, :, 0, bottom, 0] = 4.25 - bottom
        fl[:, :, :, 0, top, 0] = H - 5.75 - top
    gd, gi = _search(q, k, fl, p, dev)
    compare_topk(gd, gi, oracle.search(q, k, fl, p), p["k"])


@pytest.mark.parametrize("which", ["q", "k", "both"])
def test_pixels_with_scales_of_their_own(dev, which):
    """Pixels from 1e-12 to 1e12 in one image: each score is compared with
    the largest score its own row could have, so that a lost low-magnitude
    pixel would show (seven roundings of sums of at most that size: 4.2e-7)."""
    p = small_params(T=2, C=24, H=30, W=33, ws=5, wt=1, ps=1, k=33)
    rng = np.random.default_rng(77)
    shp = (1, 2, 24, 30, 33)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    mag = (10.0 ** rng.integers(-12, 13, (1, 2, 1, 30, 33))).astype(np.float32)
    if which != "k":
        q = q * mag
    if which != "q":
        k = k * mag
    fl = rng.integers(-2, 3, (1, 2, 2, 2, 30, 33)).astype(np.float32)
    gd, gi = _search(q, k, fl, p, dev)
    res = oracle.search(q, k, fl, p)
    ref = res["dists"][:, :33]
    fin = np.isfinite(ref)
    assert np.array_equal(fin, np.isfinite(gd))
    err = np.abs(np.where(fin, gd, 0.0) - np.where(fin, ref, 0.0))
    # |q| |k~| of the candidate bounds the sum of its products' magnitudes
    qn = np.sqrt((q.astype(np.float64) ** 2).sum(2)).reshape(-1)
    kn = np.sqrt((k.astype(np.float64) ** 2).sum(2))[0]
    y, x = np.mgrid[0:30, 0:33]
    at = gi.reshape(2, 30, 33, 33, 3)
    f = at[..., 0].astype(int)
    Y = np.clip(y[None, :, :, None] + at[..., 1], 0, 29).astype(int)
    X = np.clip(x[None, :, :, None] + at[..., 2], 0, 32).astype(int)
    bound = qn[:, None] * kn[np.clip(f, 0, 1), Y, X].reshape(-1, 33)
    assert (err <= 4.2e-7 * bound + 1e-30)[fin].all()


def _exact_scores(q, k, ps, ws):
    """64-bit scores (H, W, ws * ws) of one frame matched with itself at whole shifts, -inf outside the frame."""
    C, H, W = q.shape
    r, lo, m = ws // 2, ps // 2, ws + ps
    kp = np.pad(k.astype(np.float64), ((0, 0), (m, m), (m, m)))
    out = np.full((H, W, ws * ws), -np.inf)
    y, x = np.mgrid[0:H, 0:W]
    for d in range(ws * ws):
        dy, dx = d // ws - r, d % ws - r
        pr = np.pad((q.astype(np.float64) * kp[:, m + dy:m + dy + H, m + dx:m + dx + W]).sum(0), m)
        box = sum(pr[m - lo + a:m - lo + a + H, m - lo + b:m - lo + b + W] for a in range(ps) for b in range(ps))
        ok = (y + dy >= 0) & (y + dy < H) & (x + dx >= 0) & (x + dx < W)
        out[..., d] = np.where(ok, box, -np.inf)
    return out


@pytest.mark.parametrize("ps,C,ws", [(3, 32, 5), (1, 32, 3), (7, 64, 5), (3, 160, 5)])
@pytest.mark.parametrize("kind,bits", [("noise", 0), ("spread", 0), ("spread", 16), ("spread", 20), ("spread", 30),
                                       ("apart", 16), ("apart", 20), ("apart", 30)])
def test_error_no_larger_than_the_vector_units(dev, ps, C, ws, kind, bits):
    """Channels of q and k up to 2^bits apart (spread: falling in q, rising in
    k; apart: each has its own large channel, which the other lacks): the
    scores' error against 64 bits is no larger than that of the fp32 kernel,
    which a search that keeps every candidate runs (5% for chance)."""
    n = ws * ws
    p = small_params(T=1, C=C, H=48, W=56, ws=ws, wt=0, ps=ps, k=n)
    rng = np.random.default_rng(C + bits)
    q = rng.standard_normal((C, 48, 56))
    k = q + 0.3 * rng.standard_normal(q.shape) if kind != "noise" else rng.standard_normal(q.shape)
    if kind == "spread":
        s = 2.0 ** (-bits * np.arange(C) / (C - 1))
        q, k = q * s[:, None, None], k * s[::-1, None, None]
    elif kind == "apart":
        q[2:] *= 2.0 ** -bits
        k[2:] *= 2.0 ** -bits
        q[1] = k[0] = 0
    q, k = q.astype(np.float32), k.astype(np.float32)
    ref = _exact_scores(q, k, ps, ws)
    fl = np.zeros((1, 1, 0, 2, 48, 56), np.float32)
    gd, gi = _search(q[None, None], k[None, None], fl, p, dev)
    ad, _ = B.snls_search(torch.from_numpy(q[None, None]).to(dev), torch.from_numpy(k[None, None]).to(dev),
                          torch.from_numpy(fl).to(dev), dict(p, k=0))
    at = ((gi[..., 1] + ws // 2) * ws + gi[..., 2] + ws // 2).astype(int)
    ref = ref.reshape(-1, n)
    gref = np.take_along_axis(ref, at, 1)
    ad = ad.cpu().numpy().reshape(-1, n)
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(gd), np.isfinite(gref)) and np.array_equal(np.isfinite(ad), fin)
    rel = lambda a, b, m: np.linalg.norm(a[m].astype(np.float64) - b[m]) / np.linalg.norm(b[m])
    here, vector = rel(gd, gref, np.isfinite(gref)), rel(ad, ref, fin)
    assert here <= 1.05 * vector, (here, vector)


@pytest.mark.parametrize("ps,C,HD,ws,s1", [(3, 16, 2, 5, 0.5), (3, 32, 2, 9, 0.75), (7, 64, 1, 9, 0.5)])
def test_error_at_fractional_steps(dev, ps, C, HD, ws, s1):
    """Fractional offsets and key strides (the paper's code example: two heads
    of 8 channels, P = 3, half-pixel steps): the kept scores are no further from
    the 64-bit oracle's than the same candidates' on the vector units (5% for chance)."""
    p = small_params(T=2, C=C, HD=HD, H=40, W=44, ws=ws, wt=1, ps=ps, k=16, stride1=s1)
    rng = np.random.default_rng(C + ws)
    x = rng.standard_normal((1, 2, C, 40, 44), dtype=np.float32)
    fl = rng.uniform(-3, 3, (1, 2, 2, 2, 40, 44)).astype(np.float32)
    gd, gi = _search(x, x, fl, p, dev)
    res = oracle.search(x, x, fl, p)
    ref, ind = res["all_dists"], res["all_inds"]
    ad, ai = B.snls_search(torch.from_numpy(x).to(dev), torch.from_numpy(x).to(dev), torch.from_numpy(fl).to(dev), dict(p, k=0))
    ad = ad.cpu().numpy().reshape(ref.shape)
    assert np.array_equal(ai.cpu().numpy().reshape(ind.shape), ind.astype(np.float32))
    # the candidate of each kept position
    at = (gi[:, :, None, :] == ai.cpu().numpy().reshape(ind.shape)[:, None]).all(-1)
    assert (at.sum(-1) >= 1).all()
    at = at.argmax(-1)
    fin = np.isfinite(gd)
    exact, vector = np.take_along_axis(ref, at, 1)[fin], np.take_along_axis(ad, at, 1)[fin].astype(np.float64)
    here = np.linalg.norm(gd[fin].astype(np.float64) - exact)
    assert here <= 1.05 * np.linalg.norm(vector - exact), (here, np.linalg.norm(vector - exact))


@pytest.mark.parametrize("ps,C", [(1, 32), (3, 16), (7, 48), (3, 140)])
@pytest.mark.parametrize("what", ["nan", "inf", "huge"])
def test_values_that_are_not_finite_or_overflow(dev, ps, C, what):
    """NaN and infinite features and ones that bf16 rounds to infinity,
    anywhere in the frame: a candidate is invalid when a pixel of its patch
    inside the frame gives NaN, and not for keys that only pixels outside it
    meet.  The keys' ones are in frame 1 and the queries compared in frame 0,
    half offsets away (no tap has weight 0)."""
    p = small_params(T=2, C=C, H=34, W=36, ws=5, wt=1, ps=ps, k=16)
    rng = np.random.default_rng(C)
    shp = (1, 2, C, 34, 36)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    big = {"nan": [np.nan], "inf": [np.inf, -np.inf], "huge": [3.4028e38, -3.4e38]}[what]
    if what == "huge":
        k *= 1e-3
    for a in (q,) if what == "huge" else (q, k):
        f = 0 if a is q else 1
        for _ in range(8):
            a[0, f, rng.integers(0, C), rng.integers(0, 34), rng.integers(0, 36)] = rng.choice(big)
        a[0, f, 3, 0, 5] = a[0, f, 5, 33, 35] = a[0, f, 1, 12, 0] = a[0, f, 2, 20, 35] = big[0]
    fl = (rng.integers(-3, 3, (1, 2, 2, 2, 34, 36)) + 0.5).astype(np.float32)
    gd, gi = _search(q, k, fl, p, dev)
    n = 34 * 36
    gd, ref = gd[:n], oracle.search(q, k, fl, p)["dists"][:n, :p["k"]]
    assert not np.isnan(gd).any()
    for inf in (np.inf, -np.inf):
        assert np.array_equal((gd == inf).sum(1), (ref == inf).sum(1))
    fin = np.isfinite(ref)
    scale = np.maximum(np.abs(ref), 4 * ps * ps * np.sqrt(C))
    if what == "huge":  # products that cancel: the size of the patch's largest ones
        m = np.pad(np.abs(q[0, 0].astype(np.float64)).sum(0), ps)
        lo = ps - ps // 2
        box = sum(m[lo + a:lo + a + 34, lo + b:lo + b + 36] for a in range(ps) for b in range(ps))
        scale = np.broadcast_to(box.reshape(-1, 1) * np.abs(k).max(), ref.shape)
    assert (np.abs(gd[fin].astype(np.float64) - ref[fin]) <= 1e-5 * scale[fin]).all()


@pytest.mark.parametrize("ps", [1, 3, 7])
@pytest.mark.parametrize("share", [0.002, 0.3])
def test_infinite_features_keep_their_scores(dev, ps, share):
    """Infinite features of q and k: an infinite score stays ranked and only
    NaN ones are invalid.  Offsets of halves, so that no tap has weight 0 (0 x
    inf); the oracle sums the same products, so the signs agree."""
    p = small_params(T=2, C=16, H=34, W=36, ws=5, wt=1, ps=ps, k=20 if ps > 1 else 33)
    rng = np.random.default_rng(9 + ps)
    shp = (1, 2, 16, 34, 36)
    q, k = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    for a in (q, k):  # one channel per pixel, away from the borders
        at = rng.random((2, 20, 20)) < share
        a[0, :, 3, 7:27, 8:28] = np.where(at, np.where(rng.random(at.shape) < 0.5, np.inf, -np.inf), a[0, :, 3, 7:27, 8:28])
    fl = (rng.integers(-2, 2, (1, 2, 2, 2, 34, 36)) + 0.5).astype(np.float32)
    gd, gi = _search(q, k, fl, p, dev)
    ref = oracle.search(q, k, fl, p)["dists"][:, :p["k"]]
    assert not np.isnan(gd).any()
    # rows sorted best first: the numbers of infinite ones agree
    for inf in (np.inf, -np.inf):
        assert np.array_equal((gd == inf).sum(1), (ref == inf).sum(1))
    fin = np.isfinite(ref)
    assert np.allclose(gd[fin], ref[fin], rtol=1e-5, atol=1e-5 * ps * ps * 4)


@pytest.mark.parametrize("mq,mk", [(1e-16, 1e-20), (1e30, 1e-34), (1e-34, 1e34)])
@pytest.mark.parametrize("wide", [False, True])
def test_scales_whose_product_leaves_the_range(dev, mq, mk, wide):
    """Magnitudes whose scales multiply to a denormal or to infinity on the
    way, while the scores are ordinary numbers (wide: scales per pixel)."""
    p = small_params(T=1, C=16, H=20, W=21, ws=3, wt=0, ps=3, k=9)
    rng = np.random.default_rng(4)
    shp = (1, 1, 16, 20, 21)
    q, k = (rng.standard_normal(shp) for _ in range(2))
    if wide:
        q[..., 0, 0] *= 1e-6
        k[..., 0, 0] *= 1e-6
    fl = np.zeros((1, 1, 0, 2, 20, 21), np.float32)
    gd, gi = _search((q * mq).astype(np.float32), (k * mk).astype(np.float32), fl, p, dev)
    ref = oracle.search((q * mq).astype(np.float32), (k * mk).astype(np.float32), fl, p)["dists"][:, :9]
    fin = np.isfinite(ref)
    assert np.array_equal(fin, np.isfinite(gd))
    assert np.allclose(gd[fin] / (mq * mk), ref[fin] / (mq * mk), rtol=1e-5, atol=1e-4)


@pytest.mark.parametrize("C,HD,ws,k,s0,flow", [(32, 1, 9, 10, 1, 3.0), (64, 2, 15, 16, 1, 2.0), (31, 1, 9, 16, 1, 3.0),
                                               (40, 1, 9, 17, 1, 3.0), (96, 1, 3, 16, 1, 14.0), (32, 1, 5, 9, 2, 3.0)])
def test_single_pixel_routes(dev, C, HD, ws, k, s0, flow):
    """Single-pixel patches on both sides of the rule that takes them to the
    tiled route (32 channels per head, k = 16, query stride 1)."""
    p = small_params(T=3, C=C, HD=HD, H=37, W=45, ws=ws, wt=1, ps=1, k=k, stride0=s0)
    rng = np.random.default_rng(C + k)
    shp = (1, 3, C, 37, 45)
    q, kk = (rng.standard_normal(shp, dtype=np.float32) for _ in range(2))
    fl = rng.uniform(-flow, flow, (1, 3, 2, 2, 37, 45)).astype(np.float32)
    gd, gi = _search(q, kk, fl, p, dev)
    compare_topk(gd, gi, oracle.search(q, kk, fl, p), k)


@pytest.mark.parametrize("ps,C,k,dist", [(1, 32, 10, 0), (3, 16, 12, 0), (7, 64, 12, 1), (7, 64, 12, 0)])
def test_search_without_room_for_the_split_copies(dev, ps, C, k, dist):
    """A workspace of the size the vector-unit routes use (none for single pixels)."""
    p = small_params(T=2, C=C, H=30, W=37, ws=5, wt=1, ps=ps, k=k, dist_type=dist)
    rng = np.random.default_rng(C + ps)
    q, kk = (rng.standard_normal((1, 2, C, 30, 37), dtype=np.float32) for _ in range(2))
    fl = rng.uniform(-3, 3, (1, 2, 2, 2, 30, 37)).astype(np.float32)
    full = B.snls_workspace_size(B.SNLS_OP_SEARCH, p)
    copies = 2 * ((1 * 2 * 30 * 37 * (32 if C <= 32 else 64) * 6 + 255) // 256 * 256)
    ws = torch.empty(0 if ps == 1 else (full - copies) // 4, device=dev)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)
    gd, gi = B.snls_search(d(q), d(kk), d(fl), p, workspace=ws)
    compare_topk(gd.cpu().numpy().reshape(-1, k), gi.cpu().numpy().reshape(-1, k, 3), oracle.search(q, kk, fl, p), k)
    if ps > 1:
        with pytest.raises(B.SnlsError):
            B.snls_search(d(q), d(kk), d(fl), p, workspace=ws[:-64].clone())
