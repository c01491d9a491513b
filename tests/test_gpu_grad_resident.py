"""The gradient's one-launch sweeps (8 to 20 qubits) against its passes, which a
workspace one byte short of the size asked for selects.

The sweeps use the passes' operands and order in every single-precision operation,
so E, psi_S, dE/dh and dE/dJ are equal; dE/dgamma and dE/dt add the same doubles in
another order: 2^20 x 60 summands of either sign whose sum is at worst 1e-4 of the
sum of their magnitudes leave sqrt(2^26) 2^-53 1e4 < 1e-8.
"""
import ctypes
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2608_12058_amd as qw
    assert torch.cuda.is_available()
    qw._declare_grad(qw.lib())
    return torch, qw, qw.lib()


def grad(env, n, h, J, gam, ts, x, ckpt, short):
    torch, qw, L = env
    dp = ctypes.POINTER(ctypes.c_double)
    ptr = lambda a: a.ctypes.data_as(dp)  # noqa: E731
    S = len(gam)
    nb = int(L.qw_anneal_workspace_bytes_c64(n, ptr(h), ptr(J), S, ptr(gam), ptr(ts), ckpt))
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda")
    E, psiT = ctypes.c_double(), torch.empty_like(x)
    dg, dt, dh, dJ = np.empty(S), np.empty(S), np.empty(n), np.empty(max(1, n * (n - 1) // 2))
    st = L.qw_anneal_energy_grad_c64(
        n, ptr(h), ptr(J), S, ptr(gam), ptr(ts), ctypes.c_void_p(x.data_ptr()), ctypes.c_double(2.0 ** -23), ckpt, ctypes.byref(E),
        ptr(dg), ptr(dt), ptr(dh), ptr(dJ), ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(nb - (1 if short else 0)),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream), ctypes.c_void_p(psiT.data_ptr()), None)
    assert st == 0
    return E.value, psiT.cpu().numpy(), dh, dJ, dg, dt


def instance(torch, n, S, seed):
    h, J = synth.sk_instance(n, seed)
    gam, ts = np.linspace(1.7, 0.2, S), np.full(S, 0.4)
    x = torch.as_tensor(synth.random_state(n, seed)).to(torch.complex64).cuda()
    return np.ascontiguousarray(h), np.ascontiguousarray(J), gam, ts, x


def check(a, b, what):
    assert a[0] == b[0], what
    for i in (1, 2, 3):
        assert np.array_equal(a[i], b[i]), (what, i)
    for i in (4, 5):
        assert np.linalg.norm(a[i] - b[i]) <= 1e-8 * np.linalg.norm(b[i]), (what, i)


@pytest.mark.parametrize("n", list(range(8, 21)))
def test_sweeps_equal_passes(env, n):
    """One window, windows of one vector, of seven, and every vector kept; among the
    windows are last ones that hold b_K alone."""
    h, J, gam, ts, x = instance(env[0], n, 2, 60 + n)
    for ckpt in (0, 1, 7, -1):
        print(n, ckpt, flush=True)
        check(grad(env, n, h, J, gam, ts, x, ckpt, False), grad(env, n, h, J, gam, ts, x, ckpt, True), (n, ckpt))


def test_two_threads(env):
    """Calls of two sizes on two streams at once."""
    torch = env[0]
    cases = [(13, 4), (20, 8)]
    inst = [instance(torch, n, 3, 90 + n) for n, _ in cases]
    want = [grad(env, n, *i, c, False) for (n, c), i in zip(cases, inst)]
    got = [[], []]

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(4):
                got[k].append(grad(env, cases[k][0], *inst[k], cases[k][1], False))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for k in range(2):
        assert len(got[k]) == 4
        for g in got[k]:
            for u, v in zip(g, want[k]):
                assert np.array_equal(u, v), cases[k]
