"""Betweenness centrality on sparse graphs whose vertex kernels take several rounds
per workgroup: spans of 5,120 vertices (a round and a quarter), 8,192, and the
longest, 16,384, with more than 512 workgroups. Depths and path counts exact,
centrality against the FP64 oracle."""
import numpy as np
import pytest

import graphgen
from oracle import bc as obc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [(1 << 21) + 1, (1 << 22) - 3, (1 << 23) + 16384 + 5])
@pytest.mark.parametrize("N", [5000, 1 << 20])
def test_large_spans(V, N):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra
    rng = np.random.default_rng(V % 1000 + N)
    # vertices in use: the ends of the spans' rounds, both ends of the range, and any
    ids = np.unique(np.r_[0, V - 1, V - 2, np.arange(1, 60) * 4096 % V, np.arange(1, 60) * 5120 - 1,
                          rng.integers(0, V, 20000)])
    n = ids.size
    edges = np.unique(np.stack([ids[rng.integers(0, n, 3 * n)], ids[rng.integers(0, n, 3 * n)]], axis=1), axis=0)
    edges = edges[edges[:, 0] != edges[:, 1]]
    g = graphgen.edges_to_graph(V, edges[:, 0].astype(np.int32), edges[:, 1].astype(np.int32), True, 8, "sparse")
    gt = graphgen.transpose(g)
    seg = cagra.build_segments(cagra.DeviceGraph.from_host(g), N, 8192, 16384)
    seg_t = cagra.build_segments(cagra.DeviceGraph.from_host(gt), N, 8192, 16384)
    st = cagra.BCState(seg, seg_t)
    s = int(edges[0, 0])
    st.add_source(s)
    depth, sigma, delta = obc.single_source(g, s)
    assert (depth >= 0).sum() > n // 2
    assert np.array_equal(st.depth.cpu().numpy(), depth)
    reached = depth >= 0
    assert sigma.max() < 1 << 24  # whole numbers: exact in FP32
    assert np.array_equal(st.sigma.cpu().numpy()[reached], sigma[reached].astype(np.float32))
    delta[s] = 0.0
    # positive terms: per level a sum over the out-edges and four more roundings
    tol = depth.max() * (g.out_degree.max() + 4) * 2.0 ** -24 * delta
    assert np.all(np.abs(st.bc.cpu().numpy().astype(np.float64) - delta) <= tol)
