"""Betweenness centrality where the vertex kernels' spans end inside a round, hold
many segments or lie inside one, against the FP64 oracle; depths bit-exact."""
import numpy as np
import pytest

import graphgen
from oracle import bc as obc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [1, 255, 1023, 1024, 1025, 2049, 70001])
@pytest.mark.parametrize("N", [3, 64, 1024, 30000])
def test_spans(V, N):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra
    rng = np.random.default_rng(V + N)
    E = 4 * V if V > 1 else 0
    N = max(N, -(-V // 2000))  # at most 2,000 segments
    g = graphgen.from_edge_list(V, np.stack([rng.integers(0, V, E), rng.integers(0, V, E)], axis=1).tolist())
    gt = graphgen.transpose(g)
    seg = cagra.build_segments(cagra.DeviceGraph.from_host(g), N, 64, 4096)
    seg_t = cagra.build_segments(cagra.DeviceGraph.from_host(gt), N, 64, 4096)
    sources = [0, V - 1] if V > 1 else [0]
    got, _ = cagra.betweenness(seg, seg_t, sources)
    want = obc.betweenness(g, sources)
    # FP32 sums of at most a few hundred terms per vertex and level
    assert np.allclose(got.cpu().numpy().astype(np.float64), want, rtol=2e-5, atol=1e-5 * max(1.0, want.max()))
