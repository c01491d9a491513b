"""Polynomials of few terms take the passes where a cooperative launch or the
two-orientation plan costs more than it saves, with the same results on both sides of
the line."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _h(torch, n, d, g, x):
    """(d + g sum_j X_j) x by views."""
    y = d * x
    for j in range(n):
        a, b = x.view(-1, 2, 1 << j), y.view(-1, 2, 1 << j)
        b[:, 0] += g * a[:, 1]
        b[:, 1] += g * a[:, 0]
    return y


# first degree in one launch
@pytest.mark.parametrize("prec,n,first", [(64, 18, 1), (64, 19, 7), (64, 20, 9), (128, 17, 1), (128, 18, 4), (128, 19, 5)])
def test_caller_diagonal(prec, n, first):
    import torch
    import paper_2608_12058_amd as qw
    dt, rt = (torch.complex64, torch.float32) if prec == 64 else (torch.complex128, torch.float64)
    E = torch.as_tensor(np.random.default_rng(n).standard_normal(1 << n)).to(rt).cuda()
    psi = torch.as_tensor(synth.random_state(n, n)).to(dt).cuda()
    coef = np.random.default_rng(1).standard_normal(12) + 0.5j
    gamma, c, r = 0.8, 0.3, 2.0 * n
    # float diagonal and sums: a few units of 2^-24 (2^-53) per term
    bar = 4e-6 if prec == 64 else 2e-14
    d = (E.double() - c) / r
    t0 = psi.to(torch.complex128)
    t1 = _h(torch, n, d, gamma / r, t0)
    ref = coef[0] * t0 + coef[1] * t1
    for K in range(1, first + 2):
        if K > 1:
            t0, t1 = t1, 2.0 * _h(torch, n, d, gamma / r, t1) - t0
            ref = ref + coef[K] * t1
        y, info = qw.poly_action(psi, coef[:K + 1], gamma, shift=c, radius=r, diag=E, timing=2)
        assert (info["pass_ms"][0] > 0) == (K < first), K
        err = float(torch.linalg.vector_norm(y - ref) / torch.linalg.vector_norm(ref))
        assert err <= bar, (K, err)


@pytest.mark.parametrize("K,orientations", [(1, 3), (2, 2)])
def test_28_qubits(K, orientations):
    import torch
    import paper_2608_12058_amd as qw
    n = 28
    h, J = synth.sk_instance(n, 2)
    psi = synth.plus_state_torch(n, torch.device("cuda", 0), torch.complex64)
    _, info = qw.poly_action(psi, np.ones(K + 1), 0.8, shift=0.1, radius=3.0 * n, h=h, J=J, out=psi, timing=2)
    assert sum(x > 0 for x in info["pass_ms"]) == orientations
    torch.cuda.empty_cache()
