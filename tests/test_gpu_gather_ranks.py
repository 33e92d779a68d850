"""The gather and its reduction over the neighbours against the oracle where
the kernels change layout: 4, 2 or 1 ranks side by side (4, 8 and more channels
per head), 1 to 4 blocks of 16 channels, ranks not a multiple of the ones side
by side, more records than are staged at once, 64 and 65 output channels."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_16849_amd import snls as B
from tests.parity import assert_close
from workloads import small_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,HD,ps,s0,k,cout", [
    (4, 1, 3, 1, 5, 64), (8, 2, 3, 1, 6, 65), (16, 2, 9, 1, 7, 16), (12, 1, 5, 1, 3, 128), (40, 2, 7, 1, 11, 20),
    (36, 1, 1, 2, 9, 33), (64, 1, 3, 1, 17, 5), (48, 1, 5, 2, 4, 64),
])
def test_gather_reduce_layouts(C, HD, ps, s0, k, cout):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    p = small_params(T=2, C=C, HD=HD, H=18, W=21, ws=5, wt=1, ps=ps, k=k, stride0=s0)
    rng = np.random.default_rng(C * 100 + k)
    v = rng.standard_normal((1, 2, C, 18, 21), dtype=np.float32)
    shp = B.out_shape(p)
    w = rng.standard_normal(shp, dtype=np.float32)
    w[rng.random(shp) < 0.2] = 0.0
    inds = np.empty(shp + (3,), np.float32)
    inds[..., 0] = rng.integers(0, 2, shp)
    inds[..., 1:] = rng.uniform(-4, 4, shp + (2,))
    proj = rng.standard_normal((cout, C, k), dtype=np.float32)
    to = lambda a: torch.from_numpy(a).to(dev)
    st = B.snls_gather_stacked(to(v), to(w), to(inds), p)
    out = B.snls_gather_reduce(to(v), to(w), to(inds), to(proj), p)
    torch.cuda.synchronize()
    ref = oracle.gather_stacked(v, w, inds, p)
    assert_close(st.cpu().numpy(), ref, "stacked gather")
    assert_close(out.cpu().numpy(), oracle.stacked_reduce(ref, proj, p), "gather + reduction")
