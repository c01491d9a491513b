"""Two batches of the same launch sequence in one workspace: the second must not
replay the first one's graph, whose kernels look for descriptors and items in the
places of the first batch."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_batches_that_share_a_workspace():
    import torch
    import paper_2608_12058_amd as qw

    def batch(n, seed):
        insts = []
        for i in range(6):
            h, J = synth.sk_instance(n, seed + i)
            insts.append(dict(n=n, gamma=0.8, t=1.5, h=h, J=J))
        b = qw.Batch(insts)
        for i in range(6):
            b.state(i).copy_(torch.as_tensor(synth.random_state(n, seed + i)).to(torch.complex64))
        return insts, b

    (ia, a), (ib, b) = batch(11, 10), batch(8, 30)   # one launch of six workgroups each
    assert a.ws_bytes > b.ws_bytes
    b._ws = a._ws
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    for insts, x in ((ia, a), (ib, b), (ia, a)):
        x.out_pool.zero_()
        torch.cuda.synchronize()
        qw.expm_action_batched(x, stream=stream)
        stream.synchronize()
        for i, ins in enumerate(insts):
            want, _ = qw.expm_action(x.state(i), ins["gamma"], ins["t"], h=ins["h"], J=ins["J"], tol=1e-6)
            got = x.output(i)
            err = float(torch.linalg.vector_norm(got - want) / torch.linalg.vector_norm(want))
            assert err <= 1e-5, (ins["n"], i, err)   # twice the tolerance and complex64 sums
