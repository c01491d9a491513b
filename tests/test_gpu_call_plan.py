"""The plan that the library tells against the passes that took time, and what info
reports besides: the plan with the norm monitor."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [(64, 13), (64, 20), (64, 22), (64, 24), (64, 25), (64, 27), (128, 19), (128, 20), (128, 22),
                                    (128, 24), (128, 25)])
@pytest.mark.parametrize("diag", [False, True])
@pytest.mark.parametrize("monitor", [False, True])
def test_plan_that_ran(prec, n, diag, monitor):
    import torch
    import paper_2608_12058_amd as qw
    dev = torch.device("cuda", 0)
    psi = synth.plus_state_torch(n, dev, torch.complex64 if prec == 64 else torch.complex128)
    h, J = synth.sk_instance(n, 1)
    src = dict(diag=torch.zeros(1 << n, dtype=torch.float32 if prec == 64 else torch.float64, device=dev)) if diag else dict(h=h, J=J)
    _, info = qw.expm_action(psi, 1.0, 0.2, tol=1e-6, out=psi, monitor=monitor, timing=2, **src)
    plan = qw.call_plan(n, prec, info["K"], from_tables=not diag, monitor=monitor)
    assert [x > 0 for x in info["pass_ms"]] == [p < len(plan) for p in range(4)]
    general = qw.call_plan(n, prec, info["K"], from_tables=not diag, monitor=True)
    assert info["passes"] == len(general)
    assert info["otf_mask"] == sum(1 << p for p, o in enumerate(general) if o["rebuilds"])
    torch.cuda.empty_cache()
