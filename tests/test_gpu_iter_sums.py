"""The sums of an iteration taken by the merge's last workgroup: equal, bit for
bit, to the separate reduction launch that the gather call + merge call pair
uses, at one block, at the edges of the reducing threads' passes, with blocks of
one vertex, with split blocks and without any edge; the same for the number of
changed labels. A captured iteration gives the same on every replay."""
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


def _random(V, E, seed):
    rng = np.random.default_rng(seed)
    return graphgen.from_edge_list(V, np.stack([rng.integers(0, V, E), rng.integers(0, V, E)], axis=1).tolist())


# V, E, N, B: blocks = ceil(V / B)
CASES = {"one_block": (100, 400, 64, 128),
         "one_vertex_blocks": (300, 900, 128, 1),
         "blocks_255": (255 * 4, 3000, 256, 4),
         "blocks_256": (256 * 4, 3000, 256, 4),
         "blocks_257": (257 * 4, 3000, 256, 4),
         "blocks_1025": (1025 * 2, 9000, 512, 2),
         "blocks_2051": (2051 * 2 - 1, 9000, 512, 2),
         "no_edges": (700, 0, 256, 16)}


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("bf16", [False, True])
def test_pagerank_sums_equal_separate_reduction(cagra, name, bf16):
    import torch
    V, E, N, B = CASES[name]
    g = _random(V, E, 3) if E else graphgen.from_edge_list(V, [])
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, 4096)
    a = cagra.PageRankState(dg, seg, cagra.BF16 if bf16 else cagra.F32)
    b = cagra.PageRankState(dg, seg, cagra.BF16 if bf16 else cagra.F32)
    a.ws.fill_(0x5A)  # the iteration clears what it counts with
    a.start()
    b.start()
    for _ in range(4):
        a.step()
        b.step_split()
        assert torch.equal(a.rank_now, b.rank_now)
        assert torch.equal(a.scalars_now.view(torch.int64), b.scalars_now.view(torch.int64))


def test_split_blocks_keep_the_separate_reduction(cagra):
    import torch
    # every edge ends in the first block: its entries make several work items
    rng = np.random.default_rng(1)
    V = 1 << 16
    src = rng.permutation(V)
    g = graphgen.from_edge_list(V, np.stack([np.repeat(src, 2), rng.integers(0, 512, 2 * V)], axis=1).tolist())
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, 64, 512, 4096)
    assert seg.c.max_items > seg.c.nb
    a, b = cagra.PageRankState(dg, seg), cagra.PageRankState(dg, seg)
    a.start()
    b.start()
    for _ in range(3):
        a.step()
        b.step_split()
        assert torch.equal(a.rank_now, b.rank_now)
        assert torch.equal(a.scalars_now.view(torch.int64), b.scalars_now.view(torch.int64))


@pytest.mark.parametrize("name", list(CASES))
def test_label_changes_are_counted(cagra, name):
    import torch
    V, E, N, B = CASES[name]
    g = _random(V, E, 5) if E else graphgen.from_edge_list(V, [])
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, 4096)
    ws = cagra.iter_workspace(seg)
    ws.fill_(0x5A)
    lab = [torch.randperm(V, device="cuda", dtype=torch.int32), torch.empty(V, dtype=torch.int32, device="cuda")]
    partial = torch.empty(max(seg.Q, 1), dtype=torch.int32, device="cuda")
    changed = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    for i in range(4):
        x = lab[i & 1].cpu().numpy()
        want = x.copy()
        if E:
            dst = np.repeat(np.arange(V), np.diff(g.in_offsets))
            np.minimum.at(want, dst, x[g.in_sources])
        cagra.labelprop_iter(seg, lab[i & 1], partial, lab[1 - (i & 1)], changed, ws)
        assert np.array_equal(lab[1 - (i & 1)].cpu().numpy(), want)
        assert int(changed.item()) == int((want != x).sum())


def test_captured_iterations_replay(cagra):
    import torch
    g = _random(5000, 40000, 9)
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, 1024, 16, 4096)
    want = cagra.PageRankState(dg, seg)
    want.start()
    for _ in range(4):
        want.step_split()
    st = cagra.PageRankState(dg, seg)
    st.start()
    st.step()
    st.step()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(4):
            st.step()
    for _ in range(3):
        st.ws.fill_(0x33)  # eager work between the replays
        st.start()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(st.rank[0], want.rank_now)
        assert torch.equal(st.scalars[0].view(torch.int64), want.scalars_now.view(torch.int64))
