"""The gather kernels read staged values at fixed LDS addresses, which holds as
long as they have no static LDS: the launch's check passes each of them, and
refuses a kernel that has some."""
import ctypes
import subprocess

import pytest

pytestmark = pytest.mark.gpu


def test_no_static_lds():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_1608_01362_amd import cagra
    torch.zeros(1, device="cuda")
    L = cagra.lib()
    names = [x.split()[-1] for x in subprocess.run(["nm", "-D", cagra.LIB_PATH], capture_output=True, text=True,
                                                   check=True).stdout.splitlines() if x]
    check = getattr(L, next(n for n in names if "cagra18ensure_dynamic_lds" in n))
    check.argtypes, check.restype = [ctypes.c_void_p, ctypes.c_bool], ctypes.c_int

    def address(name):
        return ctypes.addressof(ctypes.c_char.in_dll(L, name))

    gathers = [n for n in names if n.startswith(("_ZN5cagra8k_gatherI", "_ZN5cagra14k_multi_gather"))]
    assert len(gathers) > 8
    for n in gathers:
        assert check(address(n), True) == cagra.OK, n
    other = next(n for n in names if n.startswith("_ZN5cagra11k_push_plan"))  # 64 bytes of scan temporaries
    for _ in range(2):
        assert check(address(other), True) == cagra.E_INVALID
    assert check(address(other), False) == cagra.OK
