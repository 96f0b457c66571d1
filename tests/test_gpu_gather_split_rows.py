"""Gather tiles cut into parts whose rows run over many of them: rows as long as a
segment allows, alone and between short ones, and staged BF16 values with 32-bit
edge words. Integer-valued sums and minimum labels are exact in any order."""
import numpy as np
import pytest

import graphgen
from test_gpu_gather_split import cagra  # noqa: F401

pytestmark = pytest.mark.gpu


# N, tile, long rows (each with every vertex as a source), short random edges
@pytest.mark.parametrize("N,T,rows,short", [(32768, 65536, 6, 0), (32768, 65536, 2, 0), (32768, 131072, 9, 3000),
                                            (32768, 49152, 5, 40_000), (60_000, 65536, 4, 0), (60_000, 65536, 7, 9000),
                                            (40_000, 131072, 7, 200_000), (20_000, 65536, 4, 50)])
def test_long_rows(cagra, N, T, rows, short):  # noqa: F811
    import torch
    V = 3 * N + 5000
    rng = np.random.default_rng(N + rows)
    long_dst = rng.choice(V, rows, replace=False)
    src = np.r_[np.tile(np.arange(V), rows), rng.integers(0, V, short)]
    dst = np.r_[np.repeat(long_dst, V), rng.integers(0, V, short)]
    g = graphgen.edges_to_graph(V, src.astype(np.int32), dst.astype(np.int32), True, 8, "long_rows")
    seg = cagra.build_segments(cagra.DeviceGraph.from_host(g), N, 4096, T)
    edges = np.diff(seg.arrays["tile_edge"].cpu().numpy().astype(np.int64))
    assert edges.max() >= 49152 and seg.c.ntiles <= 8 * 16  # cut: a nearly empty round of tiles long enough
    d = np.repeat(np.arange(V), np.diff(g.in_offsets))
    key = (g.in_sources // N).astype(np.int64) * V + d  # rows of the buffer: (segment, destination) ascending
    uniq, inv = np.unique(key, return_inverse=True)
    assert len(uniq) == seg.Q
    x, lab = rng.integers(0, 3, V).astype(np.int32), rng.permutation(V).astype(np.int32)
    sums = np.bincount(inv, weights=x[g.in_sources], minlength=len(uniq))
    mins = np.full(len(uniq), np.iinfo(np.int32).max, dtype=np.int32)
    np.minimum.at(mins, inv, lab[g.in_sources])
    xf = torch.from_numpy(x.astype(np.float32)).cuda()
    for t, v in ((cagra.F32, xf), (cagra.BF16, xf.bfloat16().view(torch.int16))):
        out = torch.full((seg.Q,), -1.0, dtype=torch.float32, device="cuda")
        cagra.segment_gather(seg, cagra.SUM_F32, t, v, out)
        assert np.array_equal(out.cpu().numpy(), sums.astype(np.float32)), t
    out = torch.full((seg.Q,), -1, dtype=torch.int32, device="cuda")
    cagra.segment_gather(seg, cagra.MIN_I32, cagra.I32, torch.from_numpy(lab).cuda(), out)
    assert np.array_equal(out.cpu().numpy(), mins)
