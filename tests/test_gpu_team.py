"""One-launch recurrences whose common start fails: the workgroups that have started run
them together, in place, over several exponentials and by Horner's rule too; and mixed
sizes on eight streams, where one workgroup alone took forty times as long."""
import contextlib
import ctypes
import threading
import time

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

# the project's bounds for one call in each precision
BAR = {64: 1e-5, 128: 1e-12}


@contextlib.contextmanager
def patience(qw, looks):
    f = qw.lib().qw_debug_start_patience
    f.argtypes = [ctypes.c_int]
    f(looks)
    try:
        yield
    finally:
        f(-1)


def _inputs(torch, n, prec):
    h, J = synth.sk_instance(n, 80 + n)
    x = torch.as_tensor(synth.random_state(n, n)).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
    return h, J, x


@pytest.mark.parametrize("prec,n", [(64, 13), (64, 16), (64, 18), (64, 20), (128, 15), (128, 17), (128, 19)])
@pytest.mark.parametrize("looks", [0, 1, 2])
def test_team(prec, n, looks):
    import torch
    import paper_2608_12058_amd as qw
    h, J, x = _inputs(torch, n, prec)
    E = torch.as_tensor(np.random.default_rng(n).standard_normal(1 << n)).to(torch.float32 if prec == 64 else torch.float64).cuda()
    coef = np.random.default_rng(2).standard_normal(14) * 0.5 ** np.arange(14)
    runs = [lambda out: qw.expm_action(x, 0.9, 0.6, h=h, J=J, tol=BAR[prec] / 10, out=out)[0],
            lambda out: qw.expm_action(x, 0.9, 0.6, diag=E, tol=BAR[prec] / 10, out=out)[0],
            lambda out: qw.poly_action(x, coef, 0.7, basis="mono", shift=0.2, radius=4.0 * n, h=h, J=J, out=out)[0],
            lambda out: qw.anneal_cfet4(x, h, J, [0.1, 0.9], [1.0, -1.0], 0.4, steps=4, tol=BAR[prec], out=out)[0]]
    keep = x.clone()
    for k, run in enumerate(runs):
        want = run(None)
        for rep in range(3):
            with patience(qw, looks):
                got = run(x)
            err = float(torch.linalg.vector_norm(got - want) / torch.linalg.vector_norm(want))
            x.copy_(keep)
            assert err <= BAR[prec], (k, err)


def test_mixed_sizes_on_eight_streams():
    import torch
    import paper_2608_12058_amd as qw
    rows = [[(64, 12), (64, 17), (128, 19), (64, 15)], [(64, 20), (128, 11), (64, 13), (128, 16)],
            [(64, 18), (64, 18), (128, 14), (64, 19)], [(128, 17), (64, 16), (64, 20), (64, 21)]] * 2

    def make(prec, n):
        h, J, x = _inputs(torch, n, prec)
        return prec, n, h, J, x, torch.empty_like(x), qw.Workspace.for_problem(n, prec)

    work = [[make(*s) for s in row] for row in rows]
    streams = [torch.cuda.Stream() for _ in rows]

    def run(k):
        for _ in range(8):
            for prec, n, h, J, x, y, ws in work[k]:
                qw.expm_action(x, 0.9, 1.5, h=h, J=J, tol=1e-6, out=y, workspace=ws, stream=streams[k])
                streams[k].synchronize()

    for k in range(len(rows)):
        run(k)
    want = [[p[5].clone() for p in row] for row in work]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for k in range(len(rows)):
        run(k)
    one = time.perf_counter() - t0
    threads = [threading.Thread(target=run, args=(k,)) for k in range(len(rows))]
    t0 = time.perf_counter()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    all_at_once = time.perf_counter() - t0
    print(f"one after another {one:.3f} s, at once {all_at_once:.3f} s", flush=True)
    for row, w in zip(work, want):
        for p, v in zip(row, w):
            assert float(torch.linalg.vector_norm(p[5] - v) / torch.linalg.vector_norm(v)) <= BAR[64], p[:2]
    assert all_at_once <= 4 * one + 0.1
