"""PageRank at the most segments that the merge's LDS holds with the largest
blocks: merged whole by the small graphs' kernel, with split blocks, and as one
of many graphs."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [False, True])
def test_largest_block_and_segment_count(split):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra
    V, N, B = 4015 * 16, 16, 16384
    rng = np.random.default_rng(1)
    E = 200_000
    dst = rng.integers(0, V, E)
    if split:  # nearly all edges end in the last, shorter block
        V = 4015 * 24
        N = 24
        dst = np.where(rng.random(E) < 0.97, rng.integers(5 * B, V, E), rng.integers(0, V, E))
    g = graphgen.from_edge_list(V, np.stack([rng.integers(0, V, E), dst], axis=1).tolist())
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, 65536)
    assert seg.k == 4015 and (seg.c.max_items > seg.c.nb) == split
    want, _ = oracle.pagerank(g, iters=3)
    got, _, _ = cagra.pagerank(dg, seg, iters=3)
    # fixed-point sums: one FP32 rounding per vertex and iteration of ranks that add up to one
    assert float(np.abs(got.double().cpu().numpy() - want).sum()) <= 1e-6
    mp = cagra.MultiPageRank([dg], [seg])
    mp.run_eager(3)
    assert torch.equal(mp.rank_of(0), got)
