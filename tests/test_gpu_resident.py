"""The recurrence in one launch (up to 20 qubits in complex64, 19 in complex128):
every tile shape against the oracle, its one-workgroup fallback, coefficient
arrays longer than one upload, and recording into a HIP graph."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2608_12058_amd as qw
    return torch, qw


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


# relative L2 against the oracle at 1e-13: the project's bounds for each precision
BAR = {64: 1e-5, 128: 1e-12}


def _call(torch, qw, n, prec, diag, inplace, gamma=0.8, t=1.1, seed=5):
    h, J = synth.sk_instance(n, seed)
    E = oracle.energies(n, h, J)
    psi = synth.random_state(n, seed + 1)
    dt, rt = (torch.complex64, torch.float32) if prec == 64 else (torch.complex128, torch.float64)
    x = torch.as_tensor(psi).to(dt).cuda()
    out = x if inplace else None
    kw = dict(diag=torch.as_tensor(E).to(rt).cuda()) if diag else dict(h=h, J=J)
    y, info = qw.expm_action(x, gamma, t, tol=2.0 ** -23 if prec == 64 else 1e-12, out=out, **kw)
    if diag and prec == 64:
        E = E.astype(np.float32).astype(np.float64)
    ref = oracle.expm_action(n, E, gamma, t, psi, 1e-13)
    return _rel(y.cpu().numpy().astype(np.complex128), ref), info


# 1, 2: fewer amplitudes than lanes; 6-11: one workgroup; 12-15: one XCD; above: all of them
@pytest.mark.parametrize("prec,n", [(64, n) for n in (1, 2, 6, 7, 8, 11, 12, 13, 15, 16, 18, 19, 20)] +
                         [(128, n) for n in (1, 5, 6, 7, 10, 11, 12, 14, 15, 17, 18, 19)])
@pytest.mark.parametrize("diag,inplace", [(False, True), (True, False)])
def test_shapes_match_oracle(env, prec, n, diag, inplace):
    err, _ = _call(*env, n, prec, diag, inplace)
    assert err <= BAR[prec], err


@pytest.mark.parametrize("prec,n", [(64, 12), (64, 14), (64, 17), (128, 11), (128, 14)])
def test_one_workgroup_takes_over(env, prec, n):
    """With no patience for a common start (the waits still end) the last
    workgroup to leave runs the recurrence alone, in place too."""
    torch, qw = env
    lib = qw.lib()
    lib.qw_debug_start_patience.argtypes = [ctypes.c_int]
    lib.qw_debug_start_patience(0)
    try:
        err, _ = _call(torch, qw, n, prec, False, True)
    finally:
        lib.qw_debug_start_patience(-1)
    assert err <= BAR[prec], err


@pytest.mark.parametrize("n", [7, 13, 16])
@pytest.mark.parametrize("prec,K", [(64, 439), (64, 440), (64, 1000), (128, 219), (128, 220), (128, 703)])
def test_long_coefficient_arrays(env, n, prec, K):
    """Degrees at and beyond what one upload carries (440 complex64 or 220
    complex128 coefficients), complex coefficients, against the oracle."""
    torch, qw = env
    h, J = synth.sk_instance(n, 3)
    E = oracle.energies(n, h, J)
    psi = synth.random_state(n, 4)
    rng = np.random.default_rng(K)
    coef = (rng.standard_normal(K + 1) + 1j * rng.standard_normal(K + 1)) / np.arange(1, K + 2)
    x = torch.as_tensor(psi).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
    y, info = qw.poly_action(x, coef, 0.6, basis="cheb", h=h, J=J)
    c, r = info["shift_c"], info["radius_r"]
    ref = oracle.clenshaw(n, coef, (E - c) / r, 0.6 / r, psi)
    # rounding of the float diagonal moves T_k by up to k^2 2^-24 (here summed over 1/k coefficients: K 2^-24)
    bar = max(BAR[prec], 8 * K * 2.0 ** (-24 if prec == 64 else -53))
    assert _rel(y.cpu().numpy().astype(np.complex128), ref) <= bar


@pytest.mark.parametrize("prec,n", [(64, 3), (64, 11), (64, 13), (64, 18), (64, 20), (128, 9), (128, 12), (128, 17)])
@pytest.mark.parametrize("steps", [1, 2, 3, 19, 40])
def test_chained_exponentials(env, prec, n, steps):
    """An anneal's exponentials several to a launch (2, 4, 4 + 2, 4 + 32 + 2, 4 + 32
    + 32 + 12): against the same exponentials as single calls on scaled couplings."""
    torch, qw = env
    h, J = synth.sk_instance(n, 21)
    x = torch.as_tensor(synth.random_state(n, 22)).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
    T, tol = 0.9, 1e-6 if prec == 64 else 1e-11
    y, info, sizes = qw.anneal_cfet4(x, h, J, [0.2, 0.8], [1.0, -0.9], T, steps=steps, tol=tol)
    assert info["exponentials"] == 2 * steps and len(sizes) == steps
    z, t = x, 0.0
    r3 = np.sqrt(3.0)
    for hs in sizes:
        s1, s2 = (t + (0.5 - r3 / 6) * hs) / T, (t + (0.5 + r3 / 6) * hs) / T
        for w1, w2 in ((0.25 + r3 / 6, 0.25 - r3 / 6), (0.25 - r3 / 6, 0.25 + r3 / 6)):
            al = w1 * (0.2 + 0.8 * s1) + w2 * (0.2 + 0.8 * s2)
            be = w1 * (1.0 - 0.9 * s1) + w2 * (1.0 - 0.9 * s2)
            z, _ = qw.expm_action(z, be, hs, h=al * h, J=al * J, tol=0.5 * tol * hs / T)
        t += hs
    # the truncation budget of the anneal, and the rounding of as many single calls
    bar = 2 * tol + (2e-6 if prec == 64 else 1e-13)
    assert float(torch.linalg.vector_norm(y - z) / torch.linalg.vector_norm(z)) <= bar


@pytest.mark.parametrize("prec,n", [(64, 13), (64, 17), (128, 14)])
def test_one_workgroup_takes_over_a_chain(env, prec, n):
    torch, qw = env
    h, J = synth.sk_instance(n, 31)
    x = torch.as_tensor(synth.random_state(n, 32)).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
    run = lambda out: qw.anneal_cfet4(x, h, J, [0.0, 1.0], [1.0, -1.0], 0.5, steps=4, tol=1e-5, out=out)[0]  # noqa: E731
    y = run(None)
    lib = qw.lib()
    lib.qw_debug_start_patience.argtypes = [ctypes.c_int]
    lib.qw_debug_start_patience(0)
    try:
        z = run(x)   # in place
    finally:
        lib.qw_debug_start_patience(-1)
    # the same series, summed in another order
    assert float(torch.linalg.vector_norm(y - z) / torch.linalg.vector_norm(y)) <= (4e-6 if prec == 64 else 1e-13)


@pytest.mark.parametrize("n", [10, 14, 18, 20])
def test_recorded_into_a_graph(env, n):
    """A polynomial with given shift and radius on a caller diagonal records into
    a graph; replays equal the eager call (20 qubits: by passes, so to rounding)."""
    torch, qw = env
    E = torch.as_tensor(oracle.energies(n, *synth.sk_instance(n, 8)), dtype=torch.float32).cuda()
    coef = np.array([0.3, -0.2j, 0.5, 0.1 + 0.4j, -0.6])
    x = torch.as_tensor(synth.random_state(n, 9)).to(torch.complex64).cuda()
    y, ws = torch.empty_like(x), qw.Workspace.for_problem(n, 64)
    call = lambda: qw.poly_action(x, coef, 0.7, diag=E, shift=0.2, radius=4.0 * n, out=y, workspace=ws)  # noqa: E731
    call()
    torch.cuda.synchronize()
    want = y.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for k in range(3):
        x.mul_(-1.0)
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        want = -want
        assert float((y - want).norm() / want.norm()) <= 1e-6, k
