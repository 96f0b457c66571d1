"""Collaborative filtering on few gather tiles, which are cut into parts: one
step against the FP64 oracle within the FP32 summation bound, from the first
size that is cut, with rows of very different lengths and long rows over several
parts; and a workspace of one value per tile, with which the tiles stay whole."""
import numpy as np
import pytest

import graphgen
from oracle import cf
from test_gpu_cf import K, cagra, step_bound  # noqa: F401

pytestmark = pytest.mark.gpu

# users, items (log2), ratings per user, N, B, tile
CASES = [(13, 9, 17, 1 << 30, 512, 1 << 20), (13, 9, 24, 8192, 64, 65536), (16, 3, 6, 80000, 512, 16384),
         (13, 10, 24, 1000, 512, 4096), (14, 10, 20, 40000, 128, 65536)]


@pytest.mark.parametrize("us,it,ef,N,B,T", CASES)
@pytest.mark.parametrize("whole", [False, True])
def test_step(cagra, us, it, ef, N, B, T, whole):  # noqa: F811
    import torch
    g, vals, U, I = graphgen.bipartite_ratings(us, it, ef, 1)
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, T)
    sv = cagra.segment_edge_values(dg, seg, torch.from_numpy(vals).cuda())
    X0 = cf.init_factors(g.V, K, 3, scale=0.3)
    st = cagra.CFState(dg, seg, sv, torch.from_numpy(X0).cuda())
    assert (st.ws.numel() > 8 * seg.c.ntiles + 256) == (g.E >= 1 << 18 and seg.c.ntiles <= 128)
    if whole:
        st.ws = st.ws[:8 * seg.c.ntiles + 256]
    gamma, lam = 1e-4, 0.05
    st.step(gamma, lam)
    X64 = X0.astype(np.float64)
    want, sq = cf.step(g, vals, X64, gamma, lam)
    tol = step_bound(g, vals, X64, gamma) + 2.0 ** -23 * np.abs(want) + 1e-12
    assert np.all(np.abs(st.x_now.cpu().numpy().astype(np.float64) - want) <= tol)
    assert float(st.sq.item()) == pytest.approx(sq, rel=1e-5)
