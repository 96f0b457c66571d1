"""Collaborative filtering with the workspace that the library asks for and with one
value per tile: the same bits, vectors and squared error, where few tiles are
split and where none is."""
import numpy as np
import pytest

import graphgen
from test_gpu_cf import cagra  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("us,it,ef,N,B,T", [(13, 9, 24, 8192, 64, 65536), (13, 9, 17, 1 << 30, 512, 1 << 20),
                                            (14, 10, 20, 40000, 128, 4096), (10, 6, 9, 512, 64, 4096)])
def test_same_bits(cagra, us, it, ef, N, B, T):  # noqa: F811
    import torch
    g, vals, U, I = graphgen.bipartite_ratings(us, it, ef, 1)
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, T)
    sv = cagra.segment_edge_values(dg, seg, torch.from_numpy(vals).cuda())
    x0 = torch.from_numpy(np.random.default_rng(2).random((g.V, cagra.CF_FACTORS), np.float32) * 0.3).cuda()
    states = [cagra.CFState(dg, seg, sv, x0) for _ in range(3)]
    states[1].ws = states[1].ws[:8 * max(seg.c.ntiles, 1) + 256].clone()
    states[2].ws = torch.full_like(states[2].ws, 0x5A)
    states[1].x[1].fill_(float("nan"))
    for _ in range(2):
        for st in states:
            st.step(1e-4, 0.05)
        for st in states[1:]:
            assert torch.equal(st.x_now.view(torch.int32), states[0].x_now.view(torch.int32))
            assert torch.equal(st.sq.view(torch.int64), states[0].sq.view(torch.int64))
