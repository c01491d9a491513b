"""One-launch recurrences of every kind of shape (one XCD, all of them, cooperative)
from four threads and streams at once, with anneals among them: workgroups that find
the device half taken meet, or one of them runs alone, and the results hold."""
import threading

import pytest

import synth

pytestmark = pytest.mark.gpu

# the project's bounds for one call in each precision
BAR = {64: 1e-5, 128: 1e-12}
SIZES = [[(64, 12), (64, 17), (128, 19), (64, 15)], [(64, 20), (128, 11), (64, 13), (128, 16)],
         [(64, 18), (64, 18), (128, 14), (64, 19)], [(128, 17), (64, 16), (64, 20), (64, 14)]]


@pytest.mark.parametrize("anneal", [False, True])
def test_four_threads(anneal):
    import torch
    import paper_2608_12058_amd as qw

    def make(prec, n):
        h, J = synth.sk_instance(n, 70 + n)
        x = torch.as_tensor(synth.random_state(n, n)).to(torch.complex64 if prec == 64 else torch.complex128).cuda()
        return prec, n, h, J, x, torch.empty_like(x), qw.Workspace.for_problem(n, prec)

    def run(p, stream=None):
        prec, n, h, J, x, y, ws = p
        if anneal:
            qw.anneal_cfet4(x, h, J, [0.0, 1.0], [1.0, -1.0], 0.5, steps=6, tol=BAR[prec], out=y, workspace=ws, stream=stream)
        else:
            qw.expm_action(x, 0.9, 0.8, h=h, J=J, tol=BAR[prec] / 10, out=y, workspace=ws, stream=stream)

    work = [[make(*s) for s in row] for row in SIZES]
    want = []
    for row in work:
        for p in row:
            run(p)
        torch.cuda.synchronize()
        want.append([p[5].clone() for p in row])
    bad = []

    def thread(k):
        s = torch.cuda.Stream()
        for rep in range(10):
            for p in work[k]:
                run(p, s)
        s.synchronize()
        for p, w in zip(work[k], want[k]):
            err = float(torch.linalg.vector_norm(p[5] - w) / torch.linalg.vector_norm(w))
            if not err <= BAR[p[0]]:
                bad.append((p[:2], err))

    threads = [threading.Thread(target=thread, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
