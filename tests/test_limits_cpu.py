"""Limits that the host checks before any launch, without a GPU: a build workspace
smaller than the builder takes."""
import ctypes

import pytest

from test_abi_cpu import _fake_built, _graph, cagra  # noqa: F401

BUFFER = -4


@pytest.mark.parametrize("V,N", [(1000, 100), (2000, 1), (5000, 1)])  # 10 and 2,000 segments; 5,000: the sorted form
@pytest.mark.parametrize("more", [0, 1, 255, 4096])  # bytes beyond the first array
def test_build_workspace_below_the_builders_needs(cagra, V, N, more):  # noqa: F811
    """A struct that understates the workspace: an error, nothing launched."""
    E = 100_000
    g, s = _graph(cagra, V=V, E=E), _fake_built(cagra, V=V, N=N, B=100, E=E, Q=E)
    s.build_workspace_bytes = 0
    n = (s.k + 1) * 4 + more
    assert cagra.lib().cagra_build_segments(ctypes.byref(g), ctypes.byref(s), 4096, n, None) == BUFFER
