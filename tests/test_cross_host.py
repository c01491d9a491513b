"""The words by which tiles of a cluster meet (a partner that ran this round on another
XCD is never waited for), and the maps of the two-orientation plans of 22 to 28 qubits
(host code of qw_kernels.h, CPU only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_12058_amd", "csrc")


def test_words_and_maps(tmp_path):
    hipcc = next((c for c in ("/opt/rocm/bin/hipcc", shutil.which("hipcc")) if c and os.path.exists(c)), None)
    if hipcc is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "cross_checks")
    subprocess.check_call([hipcc, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"),
                           "-I", CSRC, os.path.join(ROOT, "tests", "native", "cross_checks.cpp"), "-o", exe],
                          stderr=subprocess.DEVNULL)
    assert "CROSS OK" in subprocess.check_output([exe], text=True, timeout=60)
