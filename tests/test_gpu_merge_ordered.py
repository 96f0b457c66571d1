"""Paper-order merge: workgroups of 2 to 16 waves per block (chosen from the mean
range length), blocks cut into parts by destination, subgraphs listed in windows."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu


def _by_in_degree(g):
    """The same graph with its vertices renumbered by descending in-degree."""
    indeg = np.diff(g.in_offsets)
    new = np.empty(g.V, dtype=np.int64)
    new[np.argsort(-indeg, kind="stable")] = np.arange(g.V)
    dst = np.repeat(np.arange(g.V), indeg)
    return graphgen.from_edge_list(g.V, np.stack([new[g.in_sources], new[dst]], 1))


# (N, B): mean entries per range from below 1 to thousands on either side of the
# rule's bounds 60, 160 and 384; N = 5 lists its 3,277 subgraphs in two windows
@pytest.mark.parametrize("N,B", [(5, 512), (64, 512), (256, 1024), (512, 2048), (1024, 2048), (16384, 16384),
                                 (2000, 100), (16384, 1)])
@pytest.mark.parametrize("heavy", [False, True])
def test_merge_ordered_forms(N, B, heavy):
    import torch
    from paper_1608_01362_amd import cagra
    g = graphgen.rmat_graph(14, 16, 23)
    if heavy:
        g = _by_in_degree(g)
    dg = cagra.DeviceGraph.from_host(g)
    seg = cagra.build_segments(dg, N, B, 4096)
    ref = oracle.segment(g, N, B)
    rng = np.random.default_rng(N + B)
    p = (rng.standard_normal(seg.Q) * np.exp(rng.normal(0, 3, seg.Q))).astype(np.float32)
    want = np.zeros(g.V, dtype=np.float32)  # one FP32 addition per entry, subgraphs ascending
    for s in range(ref.k):
        lo, hi = ref.seg_row_begin[s], ref.seg_row_begin[s + 1]
        want[ref.row_dst[lo:hi]] += p[lo:hi]
    pd = torch.from_numpy(p).cuda()
    out = torch.full((g.V,), 7.0, device="cuda")
    bounds = [seg.c.max_items, seg.c.nb, seg.c.nb + seg.Q // 4 + 1]  # as built, whole blocks, not tightened
    for bound in bounds:
        seg.c.max_items = bound
        cagra.merge(seg, cagra.SUM_F32, pd, out)
        assert np.array_equal(out.cpu().numpy(), want)
    q = np.abs(p)
    cagra.merge(seg, cagra.SUM_F32_COMP, torch.from_numpy(q).cuda(), out)
    exact = oracle.merge(ref, q.astype(np.float64), oracle.SUM)
    # one rounding of the sum, and the error of the compensation term (2^-24 relative per step)
    assert np.all(np.abs(out.cpu().numpy() - exact) <= 2.0 ** -23 * exact * 1.01 + 1e-38)
    li = rng.integers(-2 ** 31, 2 ** 31 - 1, seg.Q).astype(np.int32)
    oi = torch.empty(g.V, dtype=torch.int32, device="cuda")
    cagra.merge(seg, cagra.MIN_I32, torch.from_numpy(li).cuda(), oi)
    low = np.full(g.V, 2 ** 31 - 1, dtype=np.int32)
    np.minimum.at(low, ref.row_dst, li)
    assert np.array_equal(oi.cpu().numpy(), low)
