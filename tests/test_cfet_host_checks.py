"""Pointers that the anneal refuses, at every size and before any launch: states off
16-byte and workspaces off 256-byte boundaries, as in the action."""
import ctypes

import numpy as np
import pytest

import paper_2608_12058_amd as qw

_dp = ctypes.POINTER(ctypes.c_double)


# one workgroup, one XCD, all XCDs, cooperative launch, passes
@pytest.mark.parametrize("n", [3, 13, 16, 20, 22])
@pytest.mark.parametrize("name,cs", [("qw_anneal_cfet4_c64", 8), ("qw_anneal_cfet4_c128", 16)])
@pytest.mark.parametrize("psi,out,ws", [(8, 0, 0), (0, 8, 0), (0, 0, 8), (0, 0, 128), (4, 0, 0)])
def test_misaligned_pointers_are_refused(name, cs, n, psi, out, ws):
    f = getattr(qw.lib(), name)
    h, J = np.zeros(n), np.ones(n * (n - 1) // 2)
    ab = np.array([0.5, 0.5])
    ptr = lambda x: x.ctypes.data_as(_dp)  # noqa: E731
    st = f(n, ptr(h), ptr(J), ptr(ab), 1, ptr(ab), 1, ctypes.c_double(1.0), 2, ctypes.c_double(1e-6),
           ctypes.c_void_p((1 << 20) + psi), ctypes.c_void_p((1 << 24) + out), None, 0,
           ctypes.c_void_p((1 << 28) + ws), ctypes.c_size_t(1 << 40), None, None)
    assert st == qw.QW_EINVAL
    assert b"aligned" in qw.lib().qw_last_error()
