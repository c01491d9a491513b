"""What a call runs on, as the library tells it (host only): orientations cover every
bit once, and the plans of sizes at the edges are those that the kernels are written for."""
import pytest

import paper_2608_12058_amd as qw


@pytest.mark.parametrize("prec", [64, 128])
@pytest.mark.parametrize("tables", [True, False])
@pytest.mark.parametrize("monitor", [True, False])
def test_bits_are_covered_once(prec, tables, monitor):
    for n in range(1, 33):
        for K in (1, 2, 30):
            plan = qw.call_plan(n, prec, K, from_tables=tables, monitor=monitor)
            if not plan:
                assert not monitor and n <= (20 if prec == 64 else 19)
                continue
            bits = [b for o in plan for b in range(o["g0"], o["g0"] + o["h"] + o["cross"])]
            assert sorted(bits) == list(range(n)), (n, K, plan)
            assert all(o["cross"] == 0 or (n == o["g0"] + o["h"] + o["cross"] and not monitor) for o in plan)
            assert tables or not any(o["rebuilds"] for o in plan)


def _shape(*a, **k):
    return [(o["g0"], o["h"], o["cross"], o["rebuilds"]) for o in qw.call_plan(*a, **k)]


def test_sizes_at_the_edges():
    assert _shape(20, 64, 30) == [] and _shape(20, 64, 8, from_tables=False) == [(0, 12, 0, False), (12, 8, 0, False)]
    assert len(_shape(21, 64, 30)) == 2 and _shape(19, 128, 30) == [] and len(_shape(20, 128, 30)) == 2
    # the diagonal is stored at 25 qubits, rebuilt in the strided passes from 26
    assert _shape(25, 64, 30) == [(14, 10, 1, False), (0, 14, 0, False)]
    assert _shape(26, 64, 30) == [(14, 10, 2, True), (0, 14, 0, False)]
    assert _shape(28, 64, 30) == [(14, 10, 4, True), (0, 14, 0, False)]
    assert _shape(28, 64, 30, from_tables=False) == [(14, 10, 4, False), (0, 14, 0, False)]
    assert [s[3] for s in _shape(28, 64, 30, monitor=True)] == [True, False, True]
    assert len(_shape(28, 64, 1)) == 3 and len(_shape(29, 64, 30)) == 3
    assert _shape(27, 128, 30) == [(13, 10, 4, True), (0, 13, 0, True)] and len(_shape(28, 128, 30)) == 3


def test_bad_arguments():
    for a in ((0, 64, 1), (33, 64, 1), (10, 32, 1), (10, 64, 0)):
        with pytest.raises(qw.QwError):
            qw.call_plan(*a)
