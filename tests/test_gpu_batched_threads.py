"""Batches with their one-workgroup launch on the side stream, from two threads at
once, one of which captures graphs while the other launches eagerly: the outputs of
each are those of a call alone."""
import threading

import pytest

import synth

pytestmark = pytest.mark.gpu


def _batch(torch, qw, sizes, seed):
    ins = []
    for i, n in enumerate(sizes):
        h, J = synth.sk_instance(n, seed + i)
        ins.append(dict(n=n, gamma=0.9, t=0.5 + 0.1 * i, tol=1e-6, h=h, J=J))
    b = qw.Batch(ins)
    for i, n in enumerate(sizes):
        b.state(i).copy_(torch.as_tensor(synth.random_state(n, seed + i)).to(torch.complex64))
    return b


def test_captures_beside_eager_calls():
    import torch
    import paper_2608_12058_amd as qw
    # other launch sequences, so that the first thread captures anew each time
    graphed = [_batch(torch, qw, [10, 9, 14] + [11] * k + [15], 100 * k) for k in range(1, 7)]
    eager = _batch(torch, qw, [12, 8, 8, 16], 900)
    want = []
    for b in graphed + [eager]:
        qw.expm_action_batched(b, use_graph=False)
        torch.cuda.synchronize()
        want.append(b.out_pool.clone())
        b.out_pool.zero_()
    torch.cuda.synchronize()
    bad, cached = [], []

    def run(batches, wants, reps, **kw):
        s = torch.cuda.Stream()
        for _ in range(reps):
            for b, w in zip(batches, wants):
                info = qw.expm_action_batched(b, stream=s, sched=dict(concurrent=True), **kw)
                cached.append(info["graph_cached"])
                with torch.cuda.stream(s):
                    if not torch.equal(b.out_pool, w):
                        bad.append((b.count, kw))
                    b.out_pool.zero_()
                s.synchronize()

    threads = [threading.Thread(target=run, args=(graphed, want[:-1], 4), kwargs=dict(use_graph=True)),
               threading.Thread(target=run, args=([eager], want[-1:], 40), kwargs=dict(use_graph=False))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(cached) == 4 * len(graphed) + 40 and not bad, bad
