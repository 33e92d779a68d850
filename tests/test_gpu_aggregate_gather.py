"""The tiled aggregation's listed gather against the oracle where it changes
path: lanes per position (4 to 256 channels per head, and channel counts that
are not a multiple of 4), record and frame-slot capacities, and neighbours
scattered past the bin boxes, whose taps are listed one record per lane."""
import numpy as np
import pytest
import torch

import oracle
from paper_2309_16849_amd import snls as B
from tests.parity import assert_close
from workloads import small_params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,HD,ps,k,wt,s0,spread", [
    (4, 1, 3, 5, 1, 1, 2), (12, 1, 3, 10, 1, 1, 12), (40, 2, 5, 10, 2, 1, 3), (64, 1, 7, 10, 2, 1, 2),
    (68, 1, 7, 10, 1, 1, 9), (192, 1, 7, 10, 2, 1, 2), (256, 1, 3, 7, 1, 2, 20), (128, 4, 3, 12, 3, 1, 6),
    (66, 1, 3, 8, 1, 1, 3), (7, 1, 3, 8, 1, 1, 15), (16, 1, 7, 10, 3, 1, 30), (24, 1, 5, 33, 2, 2, 4),
])
def test_aggregate_gather_paths(C, HD, ps, k, wt, s0, spread):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    dev = torch.device("cuda:0")
    p = small_params(T=4, C=C, HD=HD, H=21, W=27, ws=9, wt=wt, ps=ps, k=k, stride0=s0)
    rng = np.random.default_rng(C * 10 + k)
    v = rng.standard_normal((1, 4, C, 21, 27), dtype=np.float32)
    shp = B.out_shape(p)
    d = rng.standard_normal(shp, dtype=np.float32) * 2
    inds = np.empty(shp + (3,), np.float32)
    t = np.arange(4).reshape(1, 1, 4, 1, 1, 1)
    inds[..., 0] = np.clip(t + rng.integers(-wt, wt + 1, shp), 0, 3)
    inds[..., 1:] = rng.uniform(-spread, spread, shp + (2,))
    inds[:, :, :, 0, 0, 0, 1] = 40.0  # one neighbour far outside the frame
    to = lambda a: torch.from_numpy(a).to(dev)
    out = B.snls_aggregate(to(v), to(d), to(inds), p, 0.7)
    torch.cuda.synchronize()
    assert_close(out.cpu().numpy(), oracle.aggregate(v, d, inds, p, 0.7), "aggregate")
