"""Segment builder at the edges of its two forms and of its units: up to 2,048
segments in one counting and one scattering pass, more through the sorts;
groups of 1,024 edges per wave, tiles of 8,192, chunks of up to four tiles."""
import numpy as np
import pytest

import graphgen
from test_gpu_parity import cagra, check_layout  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,N", [(20480, 10), (20481, 10), (20479, 10), (4096, 2), (4098, 2), (1024, 1), (30000, 16),
                                 (30000, 30), (40000, 40000), (70000, 35000)])
def test_segment_counts(cagra, V, N):  # noqa: F811
    check_layout(cagra, graphgen.random_graph(V, 9 * V, V + N), N, 1000, 4096)


@pytest.mark.parametrize("E", [1, 63, 64, 65, 1023, 1024, 1025, 8191, 8192, 8193, 16385])
def test_edge_counts(cagra, E):  # noqa: F811
    """One row per source below E edges: row and group starts coincide or miss by one."""
    V = 700
    e = np.arange(E)
    g = graphgen.from_edge_list(V, np.stack([(e + 1 + e // V) % V, e % V], 1)[:E])
    check_layout(cagra, g, 100, 64, 64)


def test_empty_rows_between_groups(cagra):  # noqa: F811
    """Rows of several groups, and thousands of empty rows inside one group."""
    V = 60000
    edges = [(u, 0) for u in range(1, 5000)] + [(u, 30000) for u in range(0, 3000, 3)]
    edges += [(u, 59999) for u in range(0, 20000, 2)] + [(5, v) for v in range(40000, 40010)]
    for N in (64, 4096, 60000):
        check_layout(cagra, graphgen.from_edge_list(V, edges), N, 512, 2048)


def test_many_tiles_per_chunk(cagra):  # noqa: F811
    """Enough edges for chunks of more than one tile, the last chunk partly full."""
    import torch
    g = graphgen.rmat_graph(20, 20, 5)
    dg = cagra.DeviceGraph.from_host(g)
    assert g.E > 2 * 1024 * 8192
    for N in (1000, 32768, 1 << 19):
        seg = cagra.build_segments(dg, N, 8192, 65536)
        h = seg.host()
        src = g.in_sources.astype(np.int64)
        dst = np.repeat(np.arange(g.V), np.diff(g.in_offsets))
        order = np.argsort(src // N, kind="stable")
        ss, dd = src[order], dst[order]
        start = np.ones(g.E, dtype=bool)
        start[1:] = (ss[1:] // N != ss[:-1] // N) | (dd[1:] != dd[:-1])
        top = 15 if N <= 32768 else 31
        words = h["edge_src"].view(np.uint16 if top == 15 else np.uint32).astype(np.int64)
        assert np.array_equal(words, (ss % N) | (start.astype(np.int64) << top))
        assert np.array_equal(h["row_ptr"], np.append(np.flatnonzero(start), g.E))
        assert np.array_equal(h["row_dst"], dd[start])
    del torch
