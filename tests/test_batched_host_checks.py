"""Sizes out of range in a batch are refused before they index anything (in a process of
its own, which wrote over its stack otherwise).  No kernel is launched."""
import subprocess
import sys

import pytest

CODE = """
import ctypes, sys
import numpy as np
import paper_2608_12058_amd as qw
lib = qw.lib()
qw._declare_batched(lib)
it = (qw.BatchItem * 2)()
for x in it:
    x.n, x.gamma, x.t, x.tol = 3, 1.0, 1.0, 1e-6
it[1].n = int(sys.argv[1])
hJ = np.zeros(64).ctypes.data_as(ctypes.POINTER(ctypes.c_double))
p, ws = ctypes.c_void_p(1 << 20), ctypes.c_void_p(1 << 24)
if sys.argv[2] == "call":
    st = lib.qw_expm_action_batched_c64(it, 2, hJ, p, p, 0, ws, 1 << 30, None, None, None)
else:
    st = lib.qw_batched_tune_c64(it, 2, hJ, p, p, ws, 1 << 30, None, None, None)
assert st == qw.QW_EINVAL, st
"""


@pytest.mark.parametrize("n", [0, -5, 23, -(1 << 30), 1 << 30])
@pytest.mark.parametrize("entry", ["call", "tune"])
def test_sizes_out_of_range(n, entry):
    subprocess.check_call([sys.executable, "-c", CODE, str(n), entry], timeout=120)
