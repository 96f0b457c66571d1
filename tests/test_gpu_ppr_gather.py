"""One batched personalized iteration from arbitrary contributions against FP64
sums: shares of every remainder modulo a batch and 64 edges, empty shares, rows
over many shares, both lengths of edge word, shares on both sides of 512 edges
(rows loaded ahead or not), values and buffer on both sides of 256 MB, and a
segment of 4 GiB."""
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


def _graph(kind, V, E):
    rng = np.random.default_rng(E)
    if kind == "star":  # one row
        return graphgen.from_edge_list(V, [(v, 0) for v in range(1, E + 1)])
    src, dst = rng.integers(0, V, E), (V * rng.random(E) ** 3).astype(np.int64)
    return graphgen.from_edge_list(V, np.stack([src, dst], axis=1).tolist())


# kind, V, E, N, B, tile
CASES = [("random", 40, 7, 40, 16, 64), ("random", 300, 15 * 16, 300, 64, 4096), ("random", 300, 17 * 16, 33000, 64, 4096),
         ("star", 2000, 16 * 63, 2000, 64, 4096), ("star", 2000, 16 * 64 + 1, 40000, 512, 4096),
         ("random", 500, 16 * 65, 100, 128, 64), ("random", 3000, 16 * 300, 3000, 512, 65536),
         ("random", 3000, 16 * 511, 3000, 512, 65536), ("random", 3000, 16 * 530 + 3, 40000, 512, 65536),
         ("star", 40000, 16 * 1024 + 5, 40000, 512, 65536), ("random", 70000, 900000, 40000, 512, 16384),
         ("random", 600000, 1500000, 700000, 512, 4096), ("random", 600000, 1500000, 32768, 512, 65536),
         ("random", 1000000, 2500000, 700000, 256, 65536)]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}-{c[2]}-{c[3]}" for c in CASES])
def test_sums(cagra, case):
    import torch
    kind, V, E, N, B, T = case
    g = _graph(kind, V, E)
    seg, st = _start(cagra, g, N, B, T)
    x = torch.rand((V, 64), device="cuda") ** 4
    st.contrib[0].copy_(x.reshape(-1))
    st.step(0.85)
    dst = np.repeat(np.arange(V), np.diff(g.in_offsets))
    want = torch.zeros((V, 64), dtype=torch.float64, device="cuda")
    want.index_add_(0, torch.from_numpy(dst).cuda(), x[torch.from_numpy(g.in_sources).long().cuda()].double())
    _check(st, seg, V, want)


def _start(cagra, g, N, B, T):
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, T)
    st = cagra.PPRState(dg, seg, list(range(32)) * 2)
    st.start()
    return seg, st


def _check(st, seg, V, want, rows=slice(None)):
    import torch
    restart = torch.zeros((V, 64), dtype=torch.float64, device="cuda")
    j = torch.arange(64, device="cuda")
    restart[j % 32, j] = 0.15 + 0.85 * st.scalars[0].view(64, 4)[:, 0]
    want = 0.85 * want + restart[rows]
    got = st.ranks()[rows].double()
    # positive terms: a rounding per part of a row (16 shares of a tile at most), per
    # subgraph, and four of the update
    assert torch.all((got - want).abs() <= (16 + seg.k + 4) * 2.0 ** -24 * want)


def test_segment_of_4_gib(cagra):
    import torch
    V = (1 << 24) + 3
    u = np.r_[0, 1, V - 1 - np.arange(3000)]
    g = graphgen.from_edge_list(V, [(int(s), 5 + i % 700) for i, s in enumerate(u)])
    seg, st = _start(cagra, g, V, 512, 4096)
    assert seg.k == 1
    c = st.contrib[0].view(V, 64)
    x = torch.rand((len(u), 64), device="cuda")
    c[torch.from_numpy(u).cuda()] = x
    st.step(0.85)
    want = torch.zeros((800, 64), dtype=torch.float64, device="cuda")
    want.index_add_(0, 5 + torch.arange(len(u), device="cuda") % 700, x.double())
    _check(st, seg, 800, want, slice(0, 800))


# few tiles: cut into parts that hold the rows starting in them
SPLIT = [("star", 40000, 2047, 40000, 512, 65536), ("star", 40000, 2048, 40000, 512, 65536),
         ("star", 40000, 30000, 32768, 512, 65536), ("random", 64, 2500, 64, 64, 65536),
         ("random", 700, 5000, 700, 64, 65536), ("random", 3000, 20000, 40000, 512, 65536),
         ("random", 30000, 200000, 40000, 512, 65536), ("random", 30000, 200000, 8000, 512, 16384),
         ("random", 5000, 300000, 5000, 512, 1 << 20), ("random", 60000, 900000, 32768, 128, 1 << 20)]


@pytest.mark.parametrize("case", SPLIT, ids=[f"{c[0]}-{c[1]}-{c[2]}-{c[3]}" for c in SPLIT])
def test_split_tiles(cagra, case):
    test_sums(cagra, case)


def test_split_equals_a_tile_per_part(cagra):
    """Rows of one edge: nothing is added, so the buffer of split tiles equals that of many small ones."""
    import torch
    V = 6000
    p = np.random.default_rng(1).permutation(V)
    g = graphgen.from_edge_list(V, [(int(p[i]), int(p[i - 1])) for i in range(V)])
    x = torch.randn((V, 64), device="cuda")
    out = []
    for T in (64, 65536):
        _, st = _start(cagra, g, 2500, 512, T)
        st.contrib[0].copy_(x.reshape(-1))
        st.step(0.85)
        out.append(st.ranks().clone())
    assert torch.equal(out[0], out[1])
