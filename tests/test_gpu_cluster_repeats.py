"""Clustering of graphs with repeated edges: every row keeps all of its edges, in
light rows (also more equal ids than a slot takes), in pieces and over merges."""
import numpy as np
import pytest

import graphgen
from test_gpu_cluster import cagra  # noqa: F401

pytestmark = pytest.mark.gpu

V = 45000


def _row(n, ids, seed):
    """n edges over `ids` different sources."""
    rng = np.random.default_rng(seed)
    return np.sort(rng.choice(V, ids, replace=False)[rng.integers(0, ids, n)])


@pytest.mark.parametrize("rows", [[(2, 1)], [(5, 2), (1, 1), (300, 100)] * 20, [(97, 1), (200, 2), (4096, 3)],
                                  [(4096, 1), (4095, 2000)], [(4097, 900), (8192, 1)], [(8193, 4000), (7, 3)],
                                  [(40000, 5), (16385, 9000), (3, 1)], [(20000, 1)]])
def test_rows_keep_repeated_edges(cagra, rows):  # noqa: F811
    src = [_row(n, ids, i) for i, (n, ids) in enumerate(rows)]
    off = np.zeros(V + 1, np.int32)
    off[1:len(rows) + 1] = np.cumsum([s.size for s in src])
    off[len(rows) + 1:] = off[len(rows)]
    u = np.concatenate(src).astype(np.int32)
    g = graphgen.Graph(V, off, u, np.bincount(u, minlength=V).astype(np.int32))
    out, perm, _ = cagra.cluster(cagra.DeviceGraph.from_host(g))
    perm = perm.cpu().numpy().astype(np.int64)
    inv = np.empty(V, np.int64)
    inv[perm] = np.arange(V)
    new_off, new_src = out.in_offsets.cpu().numpy(), out.in_sources.cpu().numpy()
    assert np.array_equal(np.diff(new_off), np.diff(off)[perm])
    for i in np.flatnonzero(np.diff(new_off)):
        old = u[off[perm[i]]:off[perm[i] + 1]]
        assert np.array_equal(new_src[new_off[i]:new_off[i + 1]], np.sort(inv[old])), (i, old.size)
