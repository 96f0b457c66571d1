"""One batched personalized iteration on more tiles than are cut into parts, against
FP64 sums: shares of 512 edges (rows loaded ahead) and a little less, both lengths
of edge word, values and buffer on both sides of 256 MB."""
import numpy as np
import pytest

import graphgen
from test_gpu_ppr_gather import _check, _start, cagra  # noqa: F401

pytestmark = pytest.mark.gpu

# V, E, N, tile: shares of a sixteenth of a tile
CASES = [(70_000, 2_300_001, 30_000, 16_384), (70_000, 2_300_007, 40_000, 16_384),
         (70_000, 1_300_000, 30_000, 8_704), (70_000, 1_300_000, 40_000, 8_192),
         (600_000, 2_500_013, 32_768, 16_384), (600_000, 2_500_003, 310_000, 16_384)]


@pytest.mark.parametrize("V,E,N,T", CASES)
def test_sums(cagra, V, E, N, T):  # noqa: F811
    import torch
    rng = np.random.default_rng(E)
    src, dst = rng.integers(0, V, E), (V * rng.random(E) ** 3).astype(np.int64)  # rows of very different lengths
    g = graphgen.edges_to_graph(V, src.astype(np.int32), dst.astype(np.int32), True, 8, "skewed")
    seg, st = _start(cagra, g, N, 512, T)
    assert seg.c.ntiles > 128  # no parts
    assert (g.E >= 512 * cagra.TILE_WAVES * seg.c.ntiles) == (T != 8_192)  # loaded ahead
    assert (V + seg.Q > 1 << 20) == (V == 600_000)  # past the Infinity Cache
    x = torch.rand((V, 64), device="cuda") ** 4
    st.contrib[0].copy_(x.reshape(-1))
    st.step(0.85)
    d = np.repeat(np.arange(V), np.diff(g.in_offsets))
    want = torch.zeros((V, 64), dtype=torch.float64, device="cuda")
    want.index_add_(0, torch.from_numpy(d).cuda(), x[torch.from_numpy(g.in_sources).long().cuda()].double())
    _check(st, seg, V, want)
