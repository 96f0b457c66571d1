"""Walks of the merge and of the push expansion over ranges of given lengths:
windows of 64 entries with few, many and 64 range starts, empty ranges between
them, more than 64 ranges per block, and mean lengths on both sides of the rule
that chooses the form for short ranges. Rank sums and labels are exact."""
import numpy as np
import pytest

import graphgen
from test_gpu_walk import _fixed, cagra  # noqa: F401

pytestmark = pytest.mark.gpu

B = 1024
# lengths of the ranges of every block, one per subgraph
LENGTHS = {"ones": lambda rng: np.ones(131),
           "six_or_seven": lambda rng: np.full(70, 10),
           "seven_or_eight": lambda rng: np.full(129, 9),
           "starts_at_windows": lambda rng: np.full(66, 64),
           "empty_between": lambda rng: np.tile([0, 0, 3, 1, 0, 65], 25),
           "empty_ends": lambda rng: np.r_[np.zeros(64), np.ones(63), np.zeros(65)],
           "long_after_short": lambda rng: np.r_[np.ones(65), 700, np.full(40, 2), 900, 1, 1],
           "mixed": lambda rng: rng.choice([0, 1, 2, 5, 17, 63, 64, 65, 300], 190, p=[.3, .2, .1, .1, .1, .05, .05, .05, .05]),
           "mean_95": lambda rng: np.full(65, 95),
           "mean_96": lambda rng: np.full(65, 96)}


def _graph(name, blocks):
    """The first vertex of every subgraph has edges to vertices of every block."""
    rng = np.random.default_rng(3)
    L = LENGTHS[name](rng).astype(int)
    N = blocks * B // len(L)
    V = N * len(L)
    edges = []
    for b in range(blocks):
        for s, n in enumerate(L):
            ids = np.arange(b * B, min((b + 1) * B, V))
            edges += [(s * N, d) for d in rng.choice(ids[ids != s * N], n, replace=False)]
    return graphgen.from_edge_list(V, edges), N, L


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("blocks", [1, 3])
def test_merge_walks(cagra, name, blocks):  # noqa: F811
    import torch
    g, N, L = _graph(name, blocks)
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, 4096)
    assert seg.Q == blocks * L.sum() and seg.k == len(L) and seg.c.nb == blocks
    x = (np.random.default_rng(5).random(seg.Q) * 1e-3).astype(np.float32)
    dst = seg.arrays["row_dst"][:seg.Q].cpu().numpy().astype(np.int64)
    want = np.zeros(g.V, dtype=object)
    np.add.at(want, dst, _fixed(x))
    want = (want.astype(np.int64).astype(np.float64) * 2.0 ** -56).astype(np.float32)
    z = lambda n, t: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    rank, contrib, sc = z(g.V, torch.float32), z(g.V, torch.float32), z(4, torch.float64)
    cagra.pagerank_merge(dg, seg, 1.0, cagra.F32, z(g.V, torch.float32), z(4, torch.float64),
                         torch.from_numpy(x).cuda(), rank, contrib, sc, cagra.iter_workspace(seg))
    assert np.array_equal(rank.cpu().numpy(), want)

    lab = torch.randperm(g.V, device="cuda", dtype=torch.int32)
    out, changed = torch.empty_like(lab), torch.zeros(1, dtype=torch.int32, device="cuda")
    cagra.labelprop_iter(seg, lab, torch.empty(seg.Q, dtype=torch.int32, device="cuda"), out, changed,
                         cagra.iter_workspace(seg))
    assert np.array_equal(out.cpu().numpy(), _pull(g, lab.cpu().numpy()))


@pytest.mark.parametrize("name", list(LENGTHS))
@pytest.mark.parametrize("blocks", [1, 3])
def test_push_walks(cagra, name, blocks):  # noqa: F811
    import torch
    gt, N, L = _graph(name, blocks)
    seg_t = cagra.build_segments(cagra.DeviceGraph.from_host(gt), N, B, 4096)
    g = graphgen.transpose(gt)
    lab = torch.randperm(g.V, device="cuda", dtype=torch.int32)
    out, changed = torch.empty_like(lab), torch.zeros(1, dtype=torch.int32, device="cuda")
    cagra.labelprop_push_iter(seg_t, lab, torch.empty(seg_t.Q, dtype=torch.int32, device="cuda"), out, changed,
                              cagra.push_workspace(seg_t))
    assert np.array_equal(out.cpu().numpy(), _pull(g, lab.cpu().numpy()))


def _pull(g, x):
    want = x.copy()
    np.minimum.at(want, np.repeat(np.arange(g.V), np.diff(g.in_offsets)), x[g.in_sources])
    return want
