"""C-ABI checks that need no GPU: the library loads, exports every function
include/snls.h declares, and rejects invalid arguments with the documented
status codes before touching any buffer or the device."""
import ctypes
import os
import re

import pytest
import torch

from paper_2309_16849_amd import snls as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "snls.h")
FAKE = ctypes.c_void_p(0x1000)  # never dereferenced: every call below fails validation first
BIG = 1 << 40  # workspace size argument large enough for any case below


def _declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(snls_[a-z_]+)\s*\(", text)))


@pytest.fixture(scope="module")
def lib():
    return B.load_library()


def _params(**kw):
    p = dict(B=1, T=3, C=8, H=16, W=17, HD=2, ws=3, wt=1, ps=3, stride0=1, stride1=1.0, k=4, dist_type=0)
    p.update(kw)
    return B.params_from_dict(p)


def test_exports_every_declared_function(lib):
    names = _declared_functions()
    assert set(names) == set(B.SYMBOLS)
    for n in names:
        assert hasattr(lib, n), n


def test_abi_version_and_status_strings(lib):
    assert B.snls_abi_version() == 4
    assert B.snls_status_string(0) == "ok"
    for s in range(1, 6):
        assert B.snls_status_string(s) not in ("ok", "unknown status")
    assert B.snls_status_string(99) == "unknown status"
    assert ctypes.sizeof(B.SnlsParams) == 4 * 14  # 14 four-byte fields, no padding


BAD_PARAMS = [
    dict(ws=0), dict(ps=0), dict(wt=-1), dict(stride0=0), dict(stride1=0.0), dict(stride1=-1.0),
    dict(stride1=float("nan")), dict(C=9, HD=2), dict(HD=0), dict(B=0), dict(T=0), dict(H=0), dict(W=0),
    dict(dist_type=2), dict(k=-1), dict(k=28),  # k > (2wt+1)*ws^2 = 27
]


@pytest.mark.parametrize("kw", BAD_PARAMS, ids=[str(k) for k in BAD_PARAMS])
def test_search_rejects_bad_params(lib, kw):
    prm = _params(**kw)
    st = lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, FAKE, BIG, None)
    assert st == B.SNLS_ERR_INVALID_ARG


def test_frame_side_limit(lib):
    """H or W of 1,000,000 or more is rejected: displacements of that
    magnitude must leave every frame (one cut-off for every kernel)."""
    for kw in (dict(H=1000000, W=1), dict(H=1, W=1000000)):
        prm = _params(**kw)
        st = lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, FAKE, BIG, None)
        assert st == B.SNLS_ERR_UNSUPPORTED, kw
        assert lib.snls_workspace_size(B.SNLS_OP_AGGREGATE, ctypes.byref(prm)) == ctypes.c_size_t(-1).value
    prm = _params(H=999999, W=1, ws=1, wt=0, ps=1, k=1)
    assert lib.snls_workspace_size(B.SNLS_OP_AGGREGATE, ctypes.byref(prm)) != ctypes.c_size_t(-1).value


def test_search_rejects_bad_struct_size_and_nulls(lib):
    prm = _params()
    prm.struct_size = 12
    assert lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, FAKE, BIG, None) == B.SNLS_ERR_INVALID_ARG
    prm = _params()
    assert lib.snls_search(FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, BIG, None) == B.SNLS_ERR_INVALID_ARG
    for i in range(5):
        args = [FAKE] * 5
        args[i] = None
        q, k, fl, d, ind = args
        assert lib.snls_search(q, k, fl, ctypes.byref(prm), d, ind, FAKE, BIG, None) == B.SNLS_ERR_INVALID_ARG
    # flows may be NULL when wt == 0: the call then passes validation (checked below without a device)


def test_k_limits(lib):
    prm = _params(ws=15, wt=1, k=B.SNLS_MAX_K + 1)
    assert lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, FAKE, BIG, None) == B.SNLS_ERR_UNSUPPORTED
    assert lib.snls_topk(FAKE, FAKE, 10, 500, B.SNLS_MAX_K + 1, 0, FAKE, FAKE, None) == B.SNLS_ERR_UNSUPPORTED
    for rows, nc, k, dt in ((-1, 10, 2, 0), (5, 0, 1, 0), (5, 10, 0, 0), (5, 10, 11, 0), (5, 10, 2, 3)):
        assert lib.snls_topk(FAKE, FAKE, rows, nc, k, dt, FAKE, FAKE, None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_topk(None, FAKE, 5, 10, 2, 0, FAKE, FAKE, None) == B.SNLS_ERR_INVALID_ARG


def test_aggregate_and_backward_validation(lib):
    prm = _params(k=0)  # aggregation needs k >= 1
    big = 1 << 40
    assert lib.snls_aggregate(FAKE, FAKE, FAKE, ctypes.byref(prm), 1.0, FAKE, FAKE, big, None) == B.SNLS_ERR_INVALID_ARG
    prm = _params()
    assert lib.snls_aggregate(FAKE, FAKE, FAKE, ctypes.byref(prm), float("inf"), FAKE, FAKE, big,
                              None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_aggregate(FAKE, None, FAKE, ctypes.byref(prm), 1.0, FAKE, FAKE, big, None) == B.SNLS_ERR_INVALID_ARG
    agg_need = lib.snls_workspace_size(B.SNLS_OP_AGGREGATE, ctypes.byref(prm))
    nq = 1 * 2 * 3 * 16 * 17
    assert agg_need == ((nq * 4 * 4 + 255) // 256) * 256 + 1 * 3 * 8 * 16 * 17 * 4
    assert lib.snls_aggregate(FAKE, FAKE, FAKE, ctypes.byref(prm), 1.0, FAKE, None, big, None) == B.SNLS_ERR_WORKSPACE
    assert lib.snls_aggregate(FAKE, FAKE, FAKE, ctypes.byref(prm), 1.0, FAKE, FAKE, agg_need - 1,
                              None) == B.SNLS_ERR_WORKSPACE
    need = lib.snls_workspace_size(B.SNLS_OP_BACKWARD, ctypes.byref(prm))
    al = lambda b: (b + 255) // 256 * 256
    pairs = nq * 4
    # tiles of 4 x 8 block origins, origins in [-P, H-1] x [-P, W-1]: 5 x 3 per (B, head, frame)
    nbins = 1 * 2 * 3 * ((16 - 1 + 3) // 4 + 1) * ((17 - 1 + 3) // 8 + 1)
    # G, 4 channels-last inputs, 3 accumulators; the binned dK/dV pass adds the
    # pair scalars, 32-byte pair records, pair tiles, tile counts, cursors,
    # offsets, one entry a pair and the (4+P) x (8+P) x 64 regions of both terms
    assert need == (al(pairs * 4) + 7 * al(1 * 3 * 8 * 16 * 17 * 4) + 2 * al(pairs * 4) + al(pairs * 32)
                    + al(pairs * 4) + 2 * al(nbins * 4) + al((nbins + 1) * 4) + al(pairs * 4)
                    + al(2 * nbins * 7 * 11 * 64 * 4))
    # heads wider than 64 channels take the atomic scatter path: no bin section
    wide = _params(C=130, HD=1)
    nqw = 1 * 1 * 3 * 16 * 17
    assert lib.snls_workspace_size(B.SNLS_OP_BACKWARD, ctypes.byref(wide)) == \
        al(nqw * 4 * 4) + 7 * al(1 * 3 * 130 * 16 * 17 * 4)
    args = [FAKE] * 8
    st = lib.snls_backward(*args, ctypes.byref(prm), 1.0, FAKE, FAKE, FAKE, FAKE, None, 0, None)
    assert st == B.SNLS_ERR_WORKSPACE
    st = lib.snls_backward(*args, ctypes.byref(prm), 1.0, FAKE, FAKE, FAKE, FAKE, ctypes.c_void_p(0x1104), need,
                           None)
    assert st == B.SNLS_ERR_WORKSPACE  # not 256-byte aligned
    st = lib.snls_backward(*args, ctypes.byref(prm), 1.0, FAKE, FAKE, FAKE, None, FAKE, need, None)
    assert st == B.SNLS_ERR_INVALID_ARG  # grad_flows required when wt > 0
    assert lib.snls_workspace_size(7, ctypes.byref(prm)) == ctypes.c_size_t(-1).value
    bad = _params(ws=0)
    assert lib.snls_workspace_size(B.SNLS_OP_BACKWARD, ctypes.byref(bad)) == ctypes.c_size_t(-1).value


def test_search_workspace(lib):
    """The tiled top-k path (ps <= 7, ws <= 9, any stride0, stride1 <= 1)
    scores every candidate into the workspace; other paths need none."""
    prm = _params()
    rows, ncand = 1 * 2 * 3 * 16 * 17, 3 * 3 * 3
    need = lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(prm))
    assert need == rows * ((ncand + 31) // 32 * 32) * 4  # rows padded to a multiple of 32 candidates
    # query stride 2: a query grid of 8 x 9
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(stride0=2))) == 1 * 2 * 3 * 8 * 9 * 32 * 4
    for kw in (dict(k=0), dict(stride1=1.5), dict(ps=9), dict(ws=11, k=4)):
        assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(**kw))) == 0, kw
    # single-pixel patches at query stride 2: the scores of every candidate
    # for k above 32; up to 32 the selection runs inside the scoring kernel
    p1 = _params(ps=1, stride0=2, ws=15, k=33)
    rows1 = 1 * 2 * 3 * 8 * 9
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(p1)) == rows1 * 704 * 4  # 675 padded to 704
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ps=1, stride0=2, ws=15, k=32))) == 0
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ps=1, stride0=2, ws=17, k=30))) == 0
    # at query stride 1 too: the fused single-pixel kernel up to k = 32 (no
    # workspace), the tiled scores above
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ps=1, ws=9, k=27))) == 0
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ps=1, ws=9, k=33))) == rows * 256 * 4
    # squared L2 (key stride 1): the scores, the key-norm terms, the query-norm
    # terms, five key pair planes and the query pixel-norm plane per frame and head
    plane = (rows * 32 * 4 + 255) // 256 * 256
    a256 = lambda n: (n + 255) // 256 * 256
    pairs = a256(6 * 1 * 3 * 2 * 16 * 17 * 4)
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(dist_type=1))) == \
        2 * plane + a256(rows * 4) + pairs
    # windows above 9: tiled at P = 7 (scores; for L2 also the norm terms and
    # planes), none at other patch sizes
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ws=11, ps=7))) == rows * 384 * 4
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ws=11, ps=5))) == 0
    plane11 = (rows * 384 * 4 + 255) // 256 * 256
    # (norm terms cell by cell: the planes' fp64 summed-area tables follow)
    sat = a256(5 * 1 * 3 * 2 * 17 * 18 * 8)
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ws=11, ps=7, dist_type=1))) == \
        2 * plane11 + (rows * 4 + 255) // 256 * 256 + (6 * 1 * 3 * 2 * 16 * 17 * 4 + 255) // 256 * 256 + sat
    # the same at a fractional key stride (norm terms per cell)
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(dist_type=1, stride1=0.5))) == \
        2 * plane + a256(rows * 4) + pairs + sat
    assert lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, None, BIG, None) == B.SNLS_ERR_WORKSPACE
    assert lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, FAKE, need - 1,
                           None) == B.SNLS_ERR_WORKSPACE
    assert lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, ctypes.c_void_p(0x1104), need,
                           None) == B.SNLS_ERR_WORKSPACE  # not 256-byte aligned
    assert lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(_params(ws=0))) == ctypes.c_size_t(-1).value


@pytest.mark.skipif(torch.cuda.is_available(), reason="checks the no-device error path")
def test_valid_call_without_device_reports_hip_error(lib):
    prm = _params(wt=0)
    assert lib.snls_search(FAKE, FAKE, None, ctypes.byref(prm), FAKE, FAKE, FAKE, BIG, None) == B.SNLS_ERR_HIP


def test_binding_refuses_cpu_tensors():
    p = dict(B=1, T=1, C=2, H=4, W=4, HD=1, ws=3, wt=0, ps=1, stride0=1, stride1=1.0, k=2, dist_type=0)
    x = torch.zeros(1, 1, 2, 4, 4)
    with pytest.raises(ValueError):
        B.snls_search(x, x, None, p)


def test_stacked_and_chain_validation(lib):
    prm = _params()
    need = lib.snls_workspace_size(B.SNLS_OP_AGGREGATE_STACKED, ctypes.byref(prm))
    assert need == 1 * 2 * 3 * 16 * 17 * 4 * 4  # softmax weights, rows x k
    assert lib.snls_aggregate_stacked(FAKE, FAKE, FAKE, ctypes.byref(_params(k=0)), 1.0, FAKE, FAKE, BIG,
                                      None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_aggregate_stacked(FAKE, FAKE, None, ctypes.byref(prm), 1.0, FAKE, FAKE, BIG,
                                      None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_aggregate_stacked(FAKE, FAKE, FAKE, ctypes.byref(prm), 1.0, FAKE, FAKE, need - 1,
                                      None) == B.SNLS_ERR_WORKSPACE
    for args in ((0, 3, 4, 4, 1), (1, 0, 4, 4, 1), (1, 3, 0, 4, 1), (1, 3, 4, 0, 1), (1, 3, 4, 4, -1)):
        assert lib.snls_chain_flows(FAKE, FAKE, *args, FAKE, None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_chain_flows(FAKE, None, 1, 3, 4, 4, 2, FAKE, None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_chain_flows(FAKE, FAKE, 1, 3, 4, 4, 64, FAKE, None) == B.SNLS_ERR_UNSUPPORTED


def test_aggregate_static_validation(lib):
    """The allocation-free aggregation validates like snls_aggregate and
    refuses, before touching the device, a problem whose workspace exceeds
    the library's static scratch array."""
    prm = _params(k=0)
    assert lib.snls_aggregate_static(FAKE, FAKE, FAKE, ctypes.byref(prm), 1.0, FAKE, None) == B.SNLS_ERR_INVALID_ARG
    prm = _params()
    assert lib.snls_aggregate_static(FAKE, None, FAKE, ctypes.byref(prm), 1.0, FAKE, None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_aggregate_static(FAKE, FAKE, FAKE, ctypes.byref(prm), float("nan"), FAKE,
                                     None) == B.SNLS_ERR_INVALID_ARG
    # 1 x 5 x 64 x 256 x 256 video: 84 MB transposed copy + 13 MB weights > 64 MiB
    big = _params(T=5, C=64, H=256, W=256, HD=1, ws=3, wt=1, k=10)
    need = lib.snls_workspace_size(B.SNLS_OP_AGGREGATE, ctypes.byref(big))
    assert need > B.SNLS_STATIC_SCRATCH_BYTES
    assert lib.snls_aggregate_static(FAKE, FAKE, FAKE, ctypes.byref(big), 1.0, FAKE, None) == B.SNLS_ERR_SCRATCH
    assert B.snls_status_string(B.SNLS_ERR_SCRATCH) != "unknown status"


def test_gather_and_reduce_validation(lib):
    """The example's gather with caller weights and the reduction over the k
    neighbours validate their arguments and workspaces before any device
    work; unsupported head widths and output channel counts are refused."""
    prm = _params()  # C = 8, HD = 2: 4 channels per head
    ws_g = lib.snls_workspace_size(B.SNLS_OP_GATHER_STACKED, ctypes.byref(prm))
    ws_r = lib.snls_workspace_size(B.SNLS_OP_GATHER_REDUCE, ctypes.byref(prm))
    assert ws_g == ws_r == 1 * 3 * 8 * 16 * 17 * 4  # channels-last copy of v
    # 3 channels per head: the plain gather needs no workspace, the fused pass is refused
    odd = _params(C=6, HD=2)
    assert lib.snls_workspace_size(B.SNLS_OP_GATHER_STACKED, ctypes.byref(odd)) == 0
    assert lib.snls_gather_reduce(FAKE, FAKE, FAKE, FAKE, ctypes.byref(odd), 8, FAKE, FAKE, BIG,
                                  None) == B.SNLS_ERR_UNSUPPORTED
    assert lib.snls_gather_stacked(FAKE, None, FAKE, ctypes.byref(prm), FAKE, FAKE, BIG, None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_gather_stacked(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, ws_g - 1,
                                   None) == B.SNLS_ERR_WORKSPACE
    assert lib.snls_gather_stacked(FAKE, FAKE, FAKE, ctypes.byref(_params(k=0)), FAKE, FAKE, BIG,
                                   None) == B.SNLS_ERR_INVALID_ARG
    for cout, st in ((0, B.SNLS_ERR_INVALID_ARG), (129, B.SNLS_ERR_UNSUPPORTED)):
        assert lib.snls_stacked_reduce(FAKE, FAKE, ctypes.byref(prm), cout, FAKE, None) == st
        assert lib.snls_gather_reduce(FAKE, FAKE, FAKE, FAKE, ctypes.byref(prm), cout, FAKE, FAKE, BIG, None) == st
    assert lib.snls_stacked_reduce(FAKE, None, ctypes.byref(prm), 8, FAKE, None) == B.SNLS_ERR_INVALID_ARG
    assert lib.snls_gather_reduce(FAKE, FAKE, FAKE, FAKE, ctypes.byref(prm), 8, FAKE, None, BIG,
                                  None) == B.SNLS_ERR_WORKSPACE
    wide = _params(C=160, HD=2)  # 80 channels per head
    assert lib.snls_stacked_reduce(FAKE, FAKE, ctypes.byref(wide), 8, FAKE, None) == B.SNLS_ERR_UNSUPPORTED


def test_search_accepts_a_workspace_without_the_split_copies(lib):
    """What a search needed before the matrix cores is still accepted: nothing
    for single pixels with k <= 32, the scores' part of the tiled route, and the
    strided single-pixel route needs no more than that."""
    BAD = (B.SNLS_ERR_WORKSPACE, B.SNLS_ERR_INVALID_ARG, B.SNLS_ERR_UNSUPPORTED)

    def call(prm, ws, n):
        return lib.snls_search(FAKE, FAKE, FAKE, ctypes.byref(prm), FAKE, FAKE, ws, n, None)

    if torch.cuda.is_available():
        pytest.skip("the pointers are not real")
    size = lambda prm: lib.snls_workspace_size(B.SNLS_OP_SEARCH, ctypes.byref(prm))
    p1 = _params(C=32, HD=1, ps=1, ws=9, k=10)
    assert size(p1) > 0
    for ws, n in ((None, 0), (None, BIG), (ctypes.c_void_p(256 * 4097 + 16), BIG), (FAKE, 64)):
        assert call(p1, ws, n) not in BAD
    tiled = _params(C=32, HD=1, ps=3, ws=3, k=4)
    nq = tiled.B * tiled.HD * tiled.T * tiled.H * tiled.W
    base = (nq * 32 * 4 + 255) // 256 * 256
    assert size(tiled) > base
    assert call(tiled, FAKE, base) not in BAD
    assert call(tiled, FAKE, base - 1) == B.SNLS_ERR_WORKSPACE
    assert call(tiled, None, BIG) == B.SNLS_ERR_WORKSPACE
    scored = _params(C=32, HD=1, ps=1, stride0=2, ws=9, k=33)
    nq = scored.B * scored.HD * scored.T * ((scored.H - 1) // 2 + 1) * ((scored.W - 1) // 2 + 1)
    assert size(scored) == (nq * 256 * 4 + 255) // 256 * 256
