"""Limits that the host checks before any launch, without a GPU: a build workspace
smaller than the builder takes, and more tiles or merge blocks than one launch
of 2^32 threads holds, LDS for the PageRank merge, and the workspace of a rating
step asked for before the arrays exist."""
import ctypes

import pytest

from test_abi_cpu import _fake_built, _graph, cagra  # noqa: F401

CAPACITY, BUFFER = -3, -4


@pytest.mark.parametrize("V,N", [(1000, 100), (2000, 1), (5000, 1)])  # 10 and 2,000 segments; 5,000: the sorted form
@pytest.mark.parametrize("more", [0, 1, 255, 4096])  # bytes beyond the first array
def test_build_workspace_below_the_builders_needs(cagra, V, N, more):  # noqa: F811
    """A struct that understates the workspace: an error, nothing launched."""
    E = 100_000
    g, s = _graph(cagra, V=V, E=E), _fake_built(cagra, V=V, N=N, B=100, E=E, Q=E)
    s.build_workspace_bytes = 0
    n = (s.k + 1) * 4 + more
    assert cagra.lib().cagra_build_segments(ctypes.byref(g), ctypes.byref(s), 4096, n, None) == BUFFER


MOST = 2 ** 32 // 1024 - 1


@pytest.mark.parametrize("tiles,blocks", [(MOST + 1, 10), (1, MOST + 1)])
def test_more_workgroups_than_a_launch(cagra, tiles, blocks):  # noqa: F811
    L, r = cagra.lib(), ctypes.byref
    g, s = _graph(cagra, V=blocks, E=50), _fake_built(cagra, V=blocks, N=blocks, B=1)
    s.ntiles = tiles
    gs, big = (r(g), r(s)), 1 << 40
    assert L.cagra_pagerank_iter(*gs, 0.85, -1, 0, 1, 1, 1, 1, 1, 1, 1, 4096, big, None) == CAPACITY
    assert L.cagra_pagerank_merge(*gs, 0.85, -1, 0, 1, 1, 1, 1, 1, 1, 4096, big, None) == CAPACITY
    assert L.cagra_labelprop_iter(r(s), 1, 1, 1, 1, 4096, big, None) == CAPACITY
    assert L.cagra_degree_features(*gs, 1, 4096, big, None) == CAPACITY
    assert L.cagra_learned_start(*gs, 1, 1, 1, 1, 4096, big, None) == CAPACITY
    assert L.cagra_ppr_iter(*gs, 0.85, 1, 1, 1, 1, 1, 1, 1, 1, 1, 4096, big, None) == CAPACITY
    assert L.cagra_cf_iter(*gs, 1, 0.1, 0.1, 1, 1, 2, 1, 4096, big, None) == CAPACITY
    if tiles > MOST:
        assert L.cagra_segment_gather(r(s), 0, 0, 1, 1, None) == CAPACITY
        assert L.cagra_bc_forward_level(r(s), 0, 1, 1, 1, 1, 1, 1, 4096, big, None) == CAPACITY
    s.N, s.k, s.ntiles = 20000, -(-blocks // 20000), 1
    s.max_items = max(MOST, s.nb)
    assert L.cagra_labelprop_push_iter(r(s), 1, 1, 1, 1, 4096, big, None) == CAPACITY


@pytest.mark.parametrize("k,fits", [(4015, True), (4016, False), (4055, False), (4056, False)])
def test_lds_of_the_pagerank_merge(cagra, k, fits):  # noqa: F811
    """8 B of accumulators, 8 k + 8 + 64 of ranges, and 576 bytes of static arrays in 160 KB."""
    assert (8 * 16384 + 8 * k + 72 + 576 <= 160 * 1024) == fits
    L, r = cagra.lib(), ctypes.byref
    g, s = _graph(cagra, V=8 * k, E=50), _fake_built(cagra, V=8 * k, N=8, B=16384)
    # what fits is refused for its workspace, the next thing checked
    want = BUFFER if fits else CAPACITY
    assert L.cagra_pagerank_iter(r(g), r(s), 0.85, -1, 0, 1, 1, 1, 1, 1, 1, 1, 4096, 8, None) == want
    m = cagra.CMulti()
    assert (L.cagra_multi_query(1, r(g), r(s), r(m)) == CAPACITY) == (not fits)


def test_rating_workspace_before_the_arrays(cagra):  # noqa: F811
    """The size that the query call's struct gives is the one that the step uses."""
    L, r = cagra.lib(), ctypes.byref
    s = _fake_built(cagra, V=10_000, N=5_000, B=128, E=1 << 20, Q=10_000)
    full = L.cagra_cf_workspace_bytes(r(s))
    assert full > 8 * s.ntiles + 256
    s.row_ptr = None
    assert L.cagra_cf_workspace_bytes(r(s)) == full
