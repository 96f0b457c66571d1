"""The sums of an iteration taken by the last of 2 to 64 merge blocks (65: by a launch
of their own) have the bits of the separate reduction; also replayed from a
captured graph, and for every graph of a multi-graph run."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cagra():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra as c
    c.lib()
    return c


def _graph(cagra, V, N, B, seed, tile=4096):
    rng = np.random.default_rng(seed)
    E = 6 * V
    g = graphgen.from_edge_list(V, np.stack([rng.integers(0, V, E), rng.integers(0, V, E)], axis=1).tolist())
    dg = cagra.DeviceGraph.from_host(g)
    return dg, cagra.build_segments(dg, N, B, tile)


def _equal(a, b):
    import torch
    assert torch.equal(a.rank_now, b.rank_now)
    assert torch.equal(a.scalars_now.view(torch.int64), b.scalars_now.view(torch.int64))


@pytest.mark.parametrize("nb", [2, 3, 63, 64, 65])
@pytest.mark.parametrize("B,last", [(16, 16), (16, 1), (1500, 1499)])  # vertices of a block, of the last one
@pytest.mark.parametrize("bf16", [False, True])
def test_sums_equal_separate_reduction(cagra, nb, B, last, bf16):
    V = (nb - 1) * B + last
    dg, seg = _graph(cagra, V, max(V // 5, 4), B, nb)
    assert seg.c.nb == nb and seg.c.max_items == nb
    a, b = (cagra.PageRankState(dg, seg, cagra.BF16 if bf16 else cagra.F32) for _ in range(2))
    a.start()
    b.start()
    for i in range(5):
        a.ws.fill_(0x5A + i)  # the iteration clears what it counts with
        a.step()
        b.step_split()
        _equal(a, b)


@pytest.mark.parametrize("nb", [2, 40, 64])
def test_captured_iterations_replay(cagra, nb):
    import torch
    dg, seg = _graph(cagra, nb * 100 - 7, 512, 100, nb)
    assert seg.c.nb == nb == seg.c.max_items
    want, st = cagra.PageRankState(dg, seg), cagra.PageRankState(dg, seg)
    want.start()
    for _ in range(4):
        want.step_split()
    st.start()
    st.step()
    st.step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(4):
            st.step()
    for i in range(4):
        st.ws.fill_(0x33)  # eager work between the replays
        st.start()
        if i & 1:
            torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        _equal(st, want)


@pytest.mark.parametrize("captured", [False, True])
def test_sums_of_many_graphs(cagra, captured):
    import torch
    blocks = [1, 2, 3, 63, 64, 65, 130]  # of 64 vertices
    made = [_graph(cagra, n * 64 - 3 * i, 1024, 64, n) for i, n in enumerate(blocks)]
    dgs, segs = zip(*made)
    assert [s.c.nb for s in segs] == blocks
    mp = cagra.MultiPageRank(list(dgs), list(segs))
    if captured:
        mp.capture(4)
        for _ in range(3):
            for s in mp.scalars:
                s.fill_(float("nan"))
            mp.replay()
    else:
        mp.run_eager(4)
    torch.cuda.synchronize()
    for i, (dg, seg) in enumerate(made):
        st = cagra.PageRankState(dg, seg)
        st.start()
        for _ in range(4):
            st.step_split()
        assert torch.equal(mp.rank_of(i), st.rank_now), i
        assert torch.equal(mp.scalars_of(i).view(torch.int64), st.scalars_now.view(torch.int64)), i
