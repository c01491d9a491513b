"""Calls whose tiles wait for one another from several streams and threads at once:
with four cross bits three of them can hold every CU of an XCD, and none may wait for
long.  Tiles that give up are finished by the pass that follows, bit for bit."""
import threading
import time

import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2608_12058_amd as qw
    return torch, qw


@pytest.mark.parametrize("prec,n", [(64, 25), (64, 28), (128, 24), (128, 27)])
def test_four_calls_at_once(env, prec, n):
    torch, qw = env
    dev = torch.device("cuda", 0)
    dt = torch.complex64 if prec == 64 else torch.complex128
    h, J = synth.sk_instance(n, 3)
    psi = synth.plus_state_torch(n, dev, dt)
    streams = [torch.cuda.Stream() for _ in range(4)]
    outs = [torch.empty_like(psi) for _ in streams]
    work = [qw.Workspace.for_problem(n, prec, device=dev) for _ in streams]

    def call(i, reps):
        for _ in range(reps):
            qw.expm_action(psi, 1.0, 0.2, h=h, J=J, tol=1e-6, out=outs[i], workspace=work[i], stream=streams[i])

    torch.cuda.synchronize()
    call(0, 1)
    torch.cuda.synchronize()
    want = outs[0].clone()
    t0 = time.perf_counter()
    call(0, 2)
    torch.cuda.synchronize()
    one = time.perf_counter() - t0
    threads = [threading.Thread(target=call, args=(i, 2)) for i in range(4)]
    t0 = time.perf_counter()
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    four = time.perf_counter() - t0
    print(f"n={n} c{2 * prec}: one {one:.4f} s, four {four:.4f} s", flush=True)
    for y in outs:
        assert torch.equal(y, want)
    # 31 times as long as one after another with 0.1 s of patience for each tile
    assert four <= 3 * 4 * one + 0.1
    del psi, outs, work, want
    torch.cuda.empty_cache()
