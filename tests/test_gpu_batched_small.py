"""The one-workgroup recurrence of a batch's small instances against the oracle, at
every size that it takes and at the degrees where its coefficients' blocks of 64
and its first and last terms change; several instances of one workgroup."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2608_12058_amd as qw
    assert torch.cuda.is_available()
    return torch, qw


def run(env, oracle_mod, spec):
    torch, qw = env
    insts = []
    for n, t, seed in spec:
        h, J = synth.sk_instance(n, seed)
        insts.append(dict(n=n, gamma=0.9, t=t, tol=1e-6, h=h, J=J))
    b = qw.Batch(insts)
    states = [synth.random_state(n, seed) for n, _, seed in spec]
    for i, x in enumerate(states):
        b.state(i).copy_(torch.as_tensor(x).to(torch.complex64))
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    info = qw.expm_action_batched(b, stream=stream)
    stream.synchronize()
    assert info["small_count"] == len(spec)
    for i, (n, t, seed) in enumerate(spec):
        E = oracle_mod.energies(n, insts[i]["h"], insts[i]["J"])
        want = oracle_mod.expm_action(n, E, 0.9, t, states[i], 1e-13)
        got = b.output(i).cpu().numpy().astype(np.complex128)
        # tolerance 1e-6 and up to 300 terms of complex64 rounding
        assert np.linalg.norm(got - want) <= 1e-5 * np.linalg.norm(want), (n, t)


@pytest.mark.parametrize("n", list(range(1, 14)))
def test_every_size(env, oracle_mod, n):
    run(env, oracle_mod, [(n, t, 10 * n + i) for i, t in enumerate((0.0, 0.01, 1.0, 2.6, -4.0))])


def test_workgroups_take_several(env, oracle_mod):
    """More instances than the launch has workgroups, sizes of all three shapes."""
    run(env, oracle_mod, [(13 if i % 97 == 0 else 12 if i % 31 == 0 else 3 + i % 9, 0.3 + 0.01 * (i % 40), i)
                          for i in range(600)])
