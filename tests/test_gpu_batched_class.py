"""The default tile class at 19 and 20 qubits on both sides of 2^24 amplitudes, and its
outputs against the other class."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,cls", [([20] * 15 + [18], 1), ([20] * 16, 0), ([19] * 2 + [20] * 15 + [18], 0)])
def test_default_class(sizes, cls):
    import torch
    import paper_2608_12058_amd as qw
    inst = {n: synth.sk_instance(n, n) for n in set(sizes)}
    b = qw.Batch([dict(n=n, gamma=0.9, t=0.3, tol=1e-6, h=inst[n][0], J=inst[n][1]) for n in sizes])
    for i, n in enumerate(sizes):
        b.state(i).fill_(2.0 ** (-n / 2))
    info = qw.expm_action_batched(b)
    assert info["tile_class"][20] == info["tile_class"][19] == cls and info["tile_class"][18] == 1
    torch.cuda.synchronize()
    want = b.out_pool.clone()
    qw.expm_action_batched(b, sched=dict(tile_class={n: 1 - cls for n in (19, 20)}))
    torch.cuda.synchronize()
    for i, n in enumerate(sizes):
        o, N = b.offsets[i]
        d = torch.linalg.vector_norm(b.out_pool[o:o + N] - want[o:o + N])
        assert float(d) <= 4e-6, i   # the same sums in another order, states of norm 1
