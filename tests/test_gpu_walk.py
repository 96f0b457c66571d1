"""The merge's walk over the (subgraph, block) ranges and its fixed-point
conversion: sums of arbitrary buffer values equal, bit for bit, the sums of
trunc(x * 2^56) computed with integers on the host, over range lengths from
mostly empty to many windows, more than 64 ranges per block, and shares that end
inside a window; labels take the minimum exactly."""
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


# V, E, N, B
CASES = {"mostly_empty": (4000, 1500, 8, 16),
         "one_each": (3000, 40000, 16, 64),
         "short": (5000, 200000, 64, 512),
         "k65": (65 * 32, 60000, 32, 2080),
         "k64_edge": (64 * 32, 60000, 32, 700),
         "long": (20000, 300000, 8192, 8192),
         "few": (100, 65, 100, 100)}


def _segments(cagra, name, seed=0):
    V, E, N, B = CASES[name]
    rng = np.random.default_rng(seed)
    src, dst = rng.integers(0, V, E), (V * rng.random(E) ** 2).astype(np.int64)
    g = graphgen.from_edge_list(V, np.stack([src, dst], axis=1).tolist())
    dg = cagra.DeviceGraph.from_host(g)
    return g, dg, cagra.build_segments(dg, N, B, 4096)


def _values(kind, Q, rng):
    x = (rng.random(Q) ** 8 * 0.01).astype(np.float32)
    if kind == "signed":  # mostly in [0, 64): windows with and without a value outside
        x[rng.random(Q) < 0.01] *= -1
    elif kind == "edge":
        pool = np.array([0.0, -0.0, 2.0 ** -56, 2.0 ** -57, 1.5 * 2.0 ** -56, -1.5 * 2.0 ** -56, 2.0 ** -24,
                         2.0 ** -24 * (1 + 2.0 ** -23), 1e-40, -1e-40, 1.1754944e-38], dtype=np.float32)
        x = pool[rng.integers(0, len(pool), Q)]
        # a few large ones: a block's absolute sum stays below 64
        x[rng.integers(0, Q, 12)] = np.tile(np.array([0.99999994, 1.0, -0.75, 3.0000002], dtype=np.float32), 3)
    return x


def _fixed(x):
    m, e = np.frexp(np.abs(x.astype(np.float64)))
    return np.array([(-1 if v < 0 else 1) * ((int(mm * 2 ** 53) << 64) >> (64 + 53 - 56 - int(ee)) if 53 - 56 - int(ee) > -64
                     else int(mm * 2 ** 53) << (56 + int(ee) - 53)) for v, mm, ee in zip(x.tolist(), m, e)], dtype=object)


@pytest.mark.parametrize("name", list(CASES))
@pytest.mark.parametrize("kind", ["plain", "signed", "edge"])
def test_sums_are_exact(cagra, name, kind):
    import torch
    g, dg, seg = _segments(cagra, name)
    Q, V = seg.Q, g.V
    rng = np.random.default_rng(7)
    x = _values(kind, Q, rng)
    dst = seg.arrays["row_dst"][:Q].cpu().numpy().astype(np.int64)
    want = np.zeros(V, dtype=object)
    np.add.at(want, dst, _fixed(x))
    # damping 1 and no dangling mass: the rank is the rounded sum itself
    want = (want.astype(np.int64).astype(np.float64) * 2.0 ** -56).astype(np.float32)
    z = lambda n, t: torch.zeros(n, dtype=t, device="cuda")  # noqa: E731
    rank, contrib, sc = z(V, torch.float32), z(V, torch.float32), z(4, torch.float64)
    cagra.pagerank_merge(dg, seg, 1.0, cagra.F32, z(V, torch.float32), z(4, torch.float64), torch.from_numpy(x).cuda(),
                         rank, contrib, sc, cagra.iter_workspace(seg))
    assert np.array_equal(rank.cpu().numpy(), want)
    assert sc.cpu().numpy()[3] == 0


@pytest.mark.parametrize("name", list(CASES))
def test_labels_take_the_minimum(cagra, name):
    import torch
    g, dg, seg = _segments(cagra, name, 1)
    lab = torch.randperm(g.V, device="cuda", dtype=torch.int32)
    out = torch.empty_like(lab)
    changed = torch.zeros(1, dtype=torch.int32, device="cuda")
    cagra.labelprop_iter(seg, lab, torch.empty(max(seg.Q, 1), dtype=torch.int32, device="cuda"), out, changed,
                         cagra.iter_workspace(seg))
    x = lab.cpu().numpy()
    want = x.copy()
    np.minimum.at(want, np.repeat(np.arange(g.V), np.diff(g.in_offsets)), x[g.in_sources])
    assert np.array_equal(out.cpu().numpy(), want)
    assert int(changed.item()) == int((want != x).sum())
