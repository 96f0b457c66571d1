"""Row sort of the clustering: row lengths at its limits (light rows up to 4,096
edges, pieces of 8,192, merge units of 4,096), crowded slots, empty rows, and
out-degrees that do not belong to the graph (they only steer the work)."""
import numpy as np
import pytest

import graphgen
from test_gpu_cluster import cagra, check_bit_exact  # noqa: F401

pytestmark = pytest.mark.gpu


def _graph(V, u, v):
    return graphgen.edges_to_graph(V, np.asarray(u, np.int32), np.asarray(v, np.int32), True, 8, "rows")


def _rows(V, lengths, seed):
    """Row i has lengths[i] random sources."""
    rng = np.random.default_rng(seed)
    u = [rng.choice(V - len(lengths), n, replace=False) + len(lengths) for n in lengths]
    return _graph(V, np.concatenate(u), np.repeat(np.arange(len(lengths)), lengths))


@pytest.mark.parametrize("lengths", [[4095], [4096], [4097], [8191, 8192, 8193, 1], [0, 64, 16383, 16384, 16385],
                                     [24577, 0, 0, 3], [40000, 4097, 1, 2, 3], [1] * 3000 + [4096, 4097] + [7] * 900])
def test_row_lengths(cagra, lengths):  # noqa: F811
    check_bit_exact(cagra, _rows(45000, lengths, len(lengths)))


def _band(n, width):
    v = np.repeat(np.arange(n), width)
    return _graph(n, (v + 1 + np.tile(np.arange(width), n)) % n, v)


@pytest.mark.parametrize("name", ["band", "wide_band", "star", "communities", "two_clumps", "chain"])
def test_crowded_rows(cagra, name):  # noqa: F811
    rng = np.random.default_rng(7)
    if name == "band":
        g = _band(20000, 120)
    elif name == "wide_band":
        g = _band(9000, 5000)  # heavy rows whose pieces hold neighbouring ids
    elif name == "star":
        g = _graph(70000, np.arange(1, 70000), np.zeros(69999))
    elif name == "communities":
        v = rng.integers(0, 30000, 2_000_000)
        g = _graph(30000, v // 3000 * 3000 + rng.integers(0, 3000, v.size), v)
    elif name == "two_clumps":  # ids one apart at both ends of the range
        u = np.concatenate([np.arange(300), np.arange(10 ** 6 - 300, 10 ** 6)])
        g = _graph(10 ** 6, np.tile(u, 20), np.repeat(np.arange(20) + 5000, u.size))
    else:
        g = _graph(100000, np.arange(99999), np.arange(99999) + 1)
    check_bit_exact(cagra, g)


def test_foreign_out_degrees(cagra):  # noqa: F811
    """The order of a row does not depend on what the out-degrees add up to."""
    import torch
    g = _rows(45000, [9000, 3000, 100, 0, 4097] + [50] * 2000, 3)
    dg = cagra.DeviceGraph.from_host(g)
    for deg in (np.zeros(g.V), np.full(g.V, 2 ** 31 - 1), np.arange(g.V) % 7 * 10 ** 8):
        dg.out_degree.copy_(torch.from_numpy(deg.astype(np.int32)))
        out, perm, _ = cagra.cluster(dg)
        perm = perm.cpu().numpy().astype(np.int64)
        inv = np.empty(g.V, np.int64)
        inv[perm] = np.arange(g.V)
        off, src = out.in_offsets.cpu().numpy(), out.in_sources.cpu().numpy()
        for i in np.flatnonzero(np.diff(off))[:2100]:
            old = g.in_sources[g.in_offsets[perm[i]]:g.in_offsets[perm[i] + 1]]
            assert np.array_equal(src[off[i]:off[i + 1]], np.sort(inv[old]))
