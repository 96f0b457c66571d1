"""The ordered merge with so many small blocks that one launch would have 2^32
threads, at two waves per block, or at eight workgroups of 16 waves for a block
that is split; and split blocks whose ranges take one step, several, or get a
launch of their own."""
import numpy as np
import pytest

import graphgen

pytestmark = pytest.mark.gpu


# blocks, vertices per block: 2^32 / 128 and 2^32 / (8 * 1,024), one fewer and one more
@pytest.mark.parametrize("nb,B,heavy", [(1 << 25, 1, False), ((1 << 25) + 1, 1, False), ((1 << 25) - 1, 1, False),
                                        (1 << 19, 4, True), ((1 << 19) + 3, 4, True), ((1 << 19) - 1, 4, True)])
def test_merge(nb, B, heavy):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra
    V = nb * B - B // 2  # the last block is not full
    rng = np.random.default_rng(nb)
    dst = np.r_[0, V - 1, rng.integers(0, V, 40)]
    if heavy:  # blocks whose entries exceed four times the mean
        dst = np.r_[np.repeat([0, 1, V - 1], 300), dst]
    edges = np.unique(np.stack([dst, rng.integers(0, V, dst.size)], axis=1), axis=0)
    edges = edges[edges[:, 0] != edges[:, 1]]
    off = np.zeros(V + 1, np.int32)
    off[1:] = np.cumsum(np.bincount(edges[:, 0], minlength=V))
    deg = np.bincount(edges[:, 1], minlength=V).astype(np.int32)
    g = graphgen.Graph(V, off, edges[:, 1].astype(np.int32), deg)
    seg = cagra.build_segments(cagra.DeviceGraph.from_host(g), -(-V // 4), B, 4096)
    assert seg.c.nb == nb and (seg.c.max_items > nb) == heavy
    row_dst = seg.arrays["row_dst"].cpu().numpy()
    for op, t in ((cagra.SUM_F32, torch.float32), (cagra.SUM_F32_COMP, torch.float32), (cagra.MIN_I32, torch.int32)):
        val = torch.arange(1, seg.Q + 1, device="cuda", dtype=t)  # whole numbers: the sums are exact
        out = torch.full((V,), -1, dtype=t, device="cuda")
        cagra.merge(seg, op, val, out)
        want = np.full(V, 2 ** 31 - 1 if op == cagra.MIN_I32 else 0, np.int64)
        (np.minimum if op == cagra.MIN_I32 else np.add).at(want, row_dst, np.arange(1, seg.Q + 1))
        assert torch.equal(out, torch.from_numpy(want).cuda().to(t)), op


# vertices, hot destinations, edges, N, B: ranges of a split block below the threads, waves added to
# cover them, up to four steps with many blocks, and longer ones
@pytest.mark.parametrize("V,hot,E,N,B", [(60_000, 40, 300_000, 600, 600), (60_000, 400, 900_000, 1000, 600),
                                         (300_000, 300, 2_000_000, 5000, 64), (900_000, 500, 3_000_000, 30_000, 128),
                                         (500_000, 3000, 4_000_000, 30_000, 4096), (60_000, 60_000, 400_000, 50, 300)])
def test_split_blocks(V, hot, E, N, B):
    import torch
    from paper_1608_01362_amd import cagra
    rng = np.random.default_rng(V + hot)
    dst = np.where(rng.random(E) < 0.8, rng.integers(0, hot, E), rng.integers(0, V, E))
    if hot == V:  # every block is light but one
        dst = np.where(rng.random(E) < 0.2, 7, dst)
    g = graphgen.edges_to_graph(V, rng.integers(0, V, E).astype(np.int32), dst.astype(np.int32), True, 8, "hot")
    seg = cagra.build_segments(cagra.DeviceGraph.from_host(g), N, B, 4096)
    row_dst = seg.arrays["row_dst"].cpu().numpy()
    x = rng.integers(0, 9, seg.Q)
    bounds = [seg.c.max_items, seg.c.nb, seg.c.nb + seg.c.nb // 4 + 2]  # as built, whole blocks, not tightened
    for op, t in ((cagra.SUM_F32, torch.float32), (cagra.SUM_F32_COMP, torch.float32), (cagra.MIN_I32, torch.int32)):
        want = np.full(V, 2 ** 31 - 1 if op == cagra.MIN_I32 else 0, np.int64)
        (np.minimum if op == cagra.MIN_I32 else np.add).at(want, row_dst, x)
        for seg.c.max_items in bounds:
            out = torch.full((V,), -1, dtype=t, device="cuda")
            cagra.merge(seg, op, torch.from_numpy(x).cuda().to(t), out)
            assert torch.equal(out, torch.from_numpy(want).cuda().to(t)), (op, seg.c.max_items)
