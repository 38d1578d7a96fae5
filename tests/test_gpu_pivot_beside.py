"""Pivot totals whose middle list (65 to 128 candidates) runs beside the heavy one: the same on
one stream and on two, with handoff in both lists, against the orientation traversal."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", [1, 2])
@pytest.mark.parametrize("handoff", [{}, {"handoff_after": 64, "handoff_every": 8}, {"handoff": False}])
def test_middle_list_beside_the_heavy_one(kc, scheme, handoff):
    d = kc.orient(kc.to_device(synth.erdos_renyi(400, 0.45, 5)), kc.ORDER_DEGENERACY)
    assert d.d_max > 128
    for k in (3, 5, 7):
        want = kc.count(d, k)
        for single in (False, True):
            for _ in range(3):
                assert kc.count(d, k, pivot=True, scheme=scheme, single_stream=single, **handoff) == want
    want, omega = kc.count_all(d, pivot=False, cap=16)
    for _ in range(3):
        st, got, om = kc.count_all_status(d, cap=16, scheme=scheme, **handoff)
        assert st == kc.OK and (got, om) == (want, omega)
