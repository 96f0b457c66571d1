"""Gather launches whose last round of tiles is cut into parts (2 to 16): rows
that end inside a part, at a part's border, and rows that run over several parts
or the whole tile. Integer-valued sums and minimum labels are exact, whatever the
order. Also as a multi-graph run, bit for bit equal to the single runs."""
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


def _graph(V, E, kind, seed):
    rng = np.random.default_rng(seed)
    src = rng.integers(0, V, E)
    if kind == "even":
        dst = rng.integers(0, V, E)
    elif kind == "one_row":  # one destination for everything
        dst = np.full(E, V // 3)
    else:  # "long": a few long rows between short ones
        dst = np.where(rng.random(E) < 0.7, rng.integers(0, 7, E) * (V // 8), rng.integers(0, V, E))
    return graphgen.edges_to_graph(V, src.astype(np.int32), dst.astype(np.int32), True, 1, kind)


# edges, segment size, tile length: 1 tile (16 parts); a few tiles (one or two per
# XCD: 16 parts); 10 and 17 per XCD (2 parts, whole); 35 per XCD (one round and 8
# parts); below the split length; tiles and remainders around it; deep rings
CASES = [(60000, 8192, 65536), (160000, 8192, 65536), (780000, 8192, 65536), (1300000, 32768, 65536),
         (5000000, 32768, 65536), (8600000, 32768, 65536), (17500000, 32768, 65536),
         (200000, 8192, 16384), (400000, 8192, 49152), (300000, 32768, 262144), (3000000, 32768, 131072)]


@pytest.mark.parametrize("kind", ["even", "long", "one_row"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_split_tiles(cagra, case, kind):
    import torch
    E, N, tile = case
    V = 3 * 8192 - 5
    g = _graph(V, E, kind, E)
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, 4096, tile)
    rng = np.random.default_rng(1)
    x = rng.integers(0, 3, V).astype(np.int32)
    lab = rng.permutation(V).astype(np.int32)
    h = seg.host()
    dst = np.repeat(np.arange(V), np.diff(g.in_offsets))
    s_of = g.in_sources // N
    # rows of the buffer: (segment, destination) ascending
    key = s_of.astype(np.int64) * V + dst
    uniq, inv = np.unique(key, return_inverse=True)
    assert len(uniq) == seg.Q and np.array_equal(uniq % V, h["row_dst"][:seg.Q])
    sums = np.bincount(inv, weights=x[g.in_sources], minlength=len(uniq))
    assert sums.max() < 1 << 24
    mins = np.full(len(uniq), np.iinfo(np.int32).max, dtype=np.int32)
    np.minimum.at(mins, inv, lab[g.in_sources])
    pf = torch.full((seg.Q,), -1.0, dtype=torch.float32, device="cuda")
    cagra.segment_gather(seg, cagra.SUM_F32, cagra.F32, torch.from_numpy(x.astype(np.float32)).cuda(), pf)
    assert np.array_equal(pf.cpu().numpy(), sums.astype(np.float32))
    pb = torch.full((seg.Q,), -1.0, dtype=torch.float32, device="cuda")
    cagra.segment_gather(seg, cagra.SUM_F32, cagra.BF16,
                         torch.from_numpy(x.astype(np.float32)).cuda().bfloat16().view(torch.int16), pb)
    assert torch.equal(pb, pf)
    pi = torch.full((seg.Q,), -1, dtype=torch.int32, device="cuda")
    cagra.segment_gather(seg, cagra.MIN_I32, cagra.I32, torch.from_numpy(lab).cuda(), pi)
    assert np.array_equal(pi.cpu().numpy(), mins)


@pytest.mark.parametrize("graphs", [1, 3, 20])
def test_split_tiles_of_many_graphs(cagra, graphs):
    import torch
    gs = [_graph(9000 + 100 * i, 30000 + 40000 * (i % 5), ("even", "long", "one_row")[i % 3], i) for i in range(graphs)]
    dgs = [cagra.DeviceGraph.from_host(g) for g in gs]
    segs = [cagra.build_segments(d, 16384, 4096, 65536) for d in dgs]
    mp = cagra.MultiPageRank(dgs, segs)
    mp.run_eager(5)
    for i, (d, s) in enumerate(zip(dgs, segs)):
        single, _, _ = cagra.pagerank(d, s, iters=5)
        assert torch.equal(mp.rank_of(i), single), i
