"""Sizes of one launch where its workgroups have no room: refused beforehand (1), at
the launch itself (2) or at the gradient's second sweep (3), and on a stream with
half of the compute units masked off.  They run in passes, with the same results."""
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
def refused(qw, how):
    f = qw.lib().qw_debug_refuse_groups
    f.argtypes = [ctypes.c_int]
    f(how)
    try:
        yield
    finally:
        f(0)


def rel(torch, a, b):
    return float(torch.linalg.vector_norm(a - b) / torch.linalg.vector_norm(b))


# the project's bounds for one call in each precision
BAR = {64: 1e-5, 128: 1e-12}


def _inputs(torch, n, prec):
    h, J = synth.sk_instance(n, 40 + n)
    x = torch.as_tensor(synth.random_state(n, n)).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
    return h, J, x


@pytest.mark.parametrize("prec,n", [(64, 9), (64, 12), (64, 14), (64, 17), (64, 20), (128, 11), (128, 16), (128, 19)])
@pytest.mark.parametrize("how", [1, 2])
def test_action_and_polynomial(env, prec, n, how):
    torch, qw = env
    h, J, x = _inputs(torch, n, prec)
    coef = np.array([0.3, -0.2j, 0.5, 0.1 + 0.4j, -0.6])
    act = lambda **k: qw.expm_action(x, 0.9, 0.7, h=h, J=J, tol=BAR[prec] / 10, **k)  # noqa: E731
    pol = lambda: qw.poly_action(x, coef, 0.7, shift=0.2, radius=4.0 * n, h=h, J=J)[0]  # noqa: E731
    want, want_p = act()[0], pol()
    with refused(qw, how):
        got, info = act(timing=2)
        got_p = pol()
    # the passes ran where several workgroups would have
    assert (info["pass_ms"][0] > 0) == (n > (11 if prec == 64 else 10))
    assert rel(torch, got, want) <= BAR[prec] and rel(torch, got_p, want_p) <= BAR[prec]


@pytest.mark.parametrize("prec,n", [(64, 10), (64, 13), (64, 18), (64, 20), (128, 14), (128, 18)])
@pytest.mark.parametrize("how", [1, 2])
def test_anneal(env, prec, n, how):
    torch, qw = env
    h, J, x = _inputs(torch, n, prec)
    run = lambda: qw.anneal_cfet4(x, h, J, [0.1, 0.9], [1.0, -1.0], 0.8, steps=5, tol=1e-6)[:2]  # noqa: E731
    want, wi = run()
    with refused(qw, how):
        got, gi = run()
    assert gi["terms"] == wi["terms"] and gi["exponentials"] == wi["exponentials"]
    assert rel(torch, got, want) <= BAR[prec]


@pytest.mark.parametrize("n", [9, 13, 18, 20])
@pytest.mark.parametrize("how", [1, 2, 3])
def test_gradient_in_place(env, n, how):
    """psi_S over psi0, from which a call whose second sweep is refused starts again."""
    torch, qw = env
    h, J, x = _inputs(torch, n, 64)
    out = []
    for k in (0, how):
        psi = x.clone()
        with refused(qw, k):
            E, g, _ = qw.anneal_energy_grad(h, J, [1.1, 0.4], [0.3, 0.5], psi, ckpt_every=4, psiT_out=psi)
        out.append((E, g, psi))
    (E0, g0, p0), (E1, g1, p1) = out
    # equal states and single-precision operations; dgamma and dt add doubles in another order
    assert E0 == E1 and torch.equal(p0, p1)
    assert np.array_equal(g0["h"], g1["h"]) and np.array_equal(g0["J"], g1["J"])
    for k in ("gamma", "t"):
        assert np.linalg.norm(g0[k] - g1[k]) <= 1e-8 * np.linalg.norm(g0[k])


@pytest.fixture(scope="module")
def masked(env):
    """A stream on 16 of every 32 compute units."""
    torch, _ = env
    torch.cuda.init()
    hip = ctypes.CDLL("libamdhip64.so")
    s = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*([0x0000ffff] * 8))
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(s), ctypes.c_uint32(8), mask) == 0
    return torch.cuda.ExternalStream(s.value)


@pytest.mark.parametrize("prec,n", [(64, 10), (64, 14), (64, 18), (64, 20), (64, 25), (128, 17), (128, 19), (128, 23)])
def test_masked_stream(env, masked, prec, n):
    torch, qw = env
    h, J, x = _inputs(torch, n, prec)
    want, _ = qw.expm_action(x, 0.9, 0.3, h=h, J=J, tol=BAR[prec] / 10)
    torch.cuda.synchronize()
    got, info = qw.expm_action(x, 0.9, 0.3, h=h, J=J, tol=BAR[prec] / 10, stream=masked, timing=2)
    torch.cuda.synchronize()
    assert (info["pass_ms"][0] > 0) == (n > 11)
    if n in (23, 25):
        assert info["pass_ms"][2] > 0   # three orientations: no tile waits for another
    assert rel(torch, got, want) <= BAR[prec]
