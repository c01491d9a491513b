"""One-launch recurrences whose waves give up on their partners after one look: every
amplitude that comes out finite is right, and the gradient starts again in passes."""
import contextlib
import ctypes

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2608_12058_amd as qw
    return torch, qw


@contextlib.contextmanager
def impatient(qw):
    f = qw.lib().qw_debug_wait_limit
    f.argtypes = [ctypes.c_int]
    f(1)
    try:
        yield
    finally:
        f(-1)


@pytest.mark.parametrize("prec,n", [(64, 12), (64, 15), (64, 17), (64, 20), (128, 11), (128, 16), (128, 19)])
def test_finite_amplitudes_are_right(env, prec, n):
    torch, qw = env
    h, J = synth.sk_instance(n, 7)
    x = torch.as_tensor(synth.random_state(n, n)).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
    # an amplitude is off by at most the norm of the error, the project's bound for the state's norm 1
    bar = 1e-5 if prec == 64 else 1e-12
    coef = np.array([0.4, -0.3j, 0.5])   # few terms, through which NaN does not reach every workgroup
    runs = [lambda: qw.expm_action(x, 0.9, 0.6, h=h, J=J, tol=bar / 10)[0],
            lambda: qw.poly_action(x, coef, 0.7, shift=0.2, radius=4.0 * n, h=h, J=J)[0],
            lambda: qw.anneal_cfet4(x, h, J, [0.1, 0.9], [1.0, -1.0], 0.2, steps=3, tol=bar)[0]]
    for k, run in enumerate(runs):
        want = run()
        with impatient(qw):
            for _ in range(5):
                got = run()
                ok = torch.isfinite(torch.view_as_real(got)).all(dim=1)
                assert not ok.any() or float((got - want)[ok].abs().max()) <= bar, k


@pytest.mark.parametrize("n", [12, 16, 18, 20])
def test_gradient_starts_again(env, n):
    torch, qw = env
    h, J = synth.sk_instance(n, 9)
    x = torch.as_tensor(synth.random_state(n, n)).to(torch.complex64).cuda()
    run = lambda psi: qw.anneal_energy_grad(h, J, [1.1, 0.4], [0.3, 0.5], psi, ckpt_every=4, psiT_out=psi)[:2]  # noqa: E731
    p0, p1 = x.clone(), x.clone()
    E0, g0 = run(p0)
    with impatient(qw):
        E1, g1 = run(p1)
    # equal states and single-precision operations; dgamma and dt add doubles in another order
    assert E0 == E1 and torch.equal(p0, p1)
    assert np.array_equal(g0["h"], g1["h"]) and np.array_equal(g0["J"], g1["J"])
    for k in ("gamma", "t"):
        assert np.linalg.norm(g0[k] - g1[k]) <= 1e-8 * np.linalg.norm(g0[k])
