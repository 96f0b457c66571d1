"""Clustering tiles of more edges than the short form takes (light rows of 2,000 to
4,096 edges at a tile's end) against the oracle."""
import numpy as np
import pytest

import graphgen
from oracle import cluster as oc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths", [(4096,) * 9, (4095, 3000, 1, 4096, 2049, 17, 4000), (1030, 5, 4000) * 6,
                                     (5, 4097, 3072, 3073, 8193, 4096, 2)])
def test_lengthy_tiles(lengths):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra
    rng = np.random.default_rng(len(lengths))
    V = 20000
    e = np.concatenate([np.stack([rng.permutation(V - 100)[:n] + 100, np.full(n, i)], axis=1)
                        for i, n in enumerate(lengths)])
    g = graphgen.from_edge_list(V, e.tolist())
    new, perm, hot = cagra.cluster(cagra.DeviceGraph.from_host(g))
    wperm, whot, want = oc.cluster(g)
    assert hot == whot
    assert np.array_equal(perm.cpu().numpy(), wperm)
    assert np.array_equal(new.in_offsets.cpu().numpy(), want.in_offsets)
    assert np.array_equal(new.in_sources.cpu().numpy()[:g.E], want.in_sources)
