"""The two-orientation plan of 22-28 qubits, whose strided passes take flips from
other tiles of their cluster, and the small tiles of 20-23 qubits: polynomials of low degree against torch in
complex128 (start, fused and last passes with and without cross bits, in place),
the passes that complete what a cluster left, and long series against the general
plan, which calls with the norm monitor keep."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from device_energies import energies_torch  # noqa: E402


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2608_12058_amd as qw
    qw.lib().qw_debug_start_patience.argtypes = [ctypes.c_int]
    return torch, qw


def _state(torch, n, seed, dt):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.randn(1 << n, dtype=dt, device="cuda", generator=g)
    return x / torch.linalg.vector_norm(x)


def _h(torch, n, d, g, x):
    """(d + g sum_j X_j) x by views."""
    y = d * x
    for j in range(n):
        a, b = x.view(-1, 2, 1 << j), y.view(-1, 2, 1 << j)
        b[:, 0] += g * a[:, 1]
        b[:, 1] += g * a[:, 0]
    return y


# degree 1: start pass with cross bits, last pass without; 2: a fused pass without,
# the last with; 3 and 4: a fused pass with cross bits, either ending
CASES = [(64, 25), (64, 26), (64, 28), (128, 22), (128, 23), (128, 24), (128, 26), (128, 27)]


SMALL = [(64, 21), (64, 22), (64, 23), (128, 20), (128, 21)]


@pytest.mark.parametrize("prec,n", CASES + SMALL)
@pytest.mark.parametrize("diag", [False, True])
@pytest.mark.parametrize("patience", [-1, 0])
def test_low_degrees_match_torch(env, prec, n, diag, patience):
    torch, qw = env
    dt, rt = (torch.complex64, torch.float32) if prec == 64 else (torch.complex128, torch.float64)
    h, J = synth.sk_instance(n, 60 + n)
    E = energies_torch(torch, n, h, J, torch.float64)
    if diag:
        E = E.to(rt).double()
    psi = _state(torch, n, n, dt)
    gamma, c, r = 0.8, 0.3, 2.5 * n
    coef = np.array([0.7 - 0.1j, -0.4 + 0.3j, 0.2 + 0.5j, -0.6, 0.35j])
    d = (E - c) / r
    # float diagonal and sums: a few units of 2^-24 (2^-53) per term
    bar = 2e-6 if prec == 64 else 1e-14
    t0 = psi.to(torch.complex128)
    t1 = _h(torch, n, d, gamma / r, t0)
    ref = coef[0] * t0 + coef[1] * t1
    src = dict(diag=E.to(rt)) if diag else dict(h=h, J=J)
    lib = qw.lib()
    lib.qw_debug_start_patience(patience)
    try:
        for K in range(1, 5):
            if K > 1:
                t0, t1 = t1, 2.0 * _h(torch, n, d, gamma / r, t1) - t0
                ref += coef[K] * t1
            x = psi.clone()
            y, _ = qw.poly_action(x, coef[:K + 1], gamma, shift=c, radius=r, out=x, **src)
            err = float(torch.linalg.vector_norm(y - ref) / torch.linalg.vector_norm(ref))
            assert err <= bar, (K, err)
    finally:
        lib.qw_debug_start_patience(-1)
    torch.cuda.empty_cache()


@pytest.mark.parametrize("prec,n", CASES + [(64, 27), (128, 25)])
def test_long_series_match_the_general_plan(env, prec, n):
    torch, qw = env
    dt = torch.complex64 if prec == 64 else torch.complex128
    h, J = synth.sk_instance(n, 90 + n)
    psi = _state(torch, n, n + 1, dt)
    tol = 2.0 ** -23 if prec == 64 else 1e-12
    y, _ = qw.expm_action(psi, 0.9, 0.4, h=h, J=J, tol=tol)
    z, _ = qw.expm_action(psi, 0.9, 0.4, h=h, J=J, tol=tol, monitor=True)
    err = float(torch.linalg.vector_norm(y - z) / torch.linalg.vector_norm(z))
    assert err <= (1e-5 if prec == 64 else 1e-12), err
    del y, z, psi
    torch.cuda.empty_cache()
