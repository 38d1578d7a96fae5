"""Admission of pivot queries by the LDS of the launches they make: what runs at one time stays
within the device's, several pivot queries do run at one time, and counts do not depend on it."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("smin,smax,density,lo,hi", [(40, 60, 0.9, 33, 64), (90, 110, 0.9, 65, 128), (190, 220, 0.8, 129, 256)])
def test_pivot_queries_share_the_lds(kc, smin, smax, density, lo, hi):
    import torch
    lds_dev = torch.cuda.get_device_properties(0).multi_processor_count * 160 * 1024
    g = kc.to_device(synth.dense_core(20000, 8.0, 2.1, 3, smin, smax, density, 7))
    d = kc.orient(g, kc.ORDER_DEGENERACY)
    assert lo <= d.d_max <= hi
    want = kc.count(d, 4)
    with kc.Server([d], slots=4, mem_budget=4 << 30) as sv:
        one = sv.wait(sv.submit(0, 4, True))
        rs = [sv.wait(t) for t in [sv.submit(0, 4, True) for _ in range(12)]]
    assert all(r.status == kc.OK and r.value == want for r in rs + [one])
    # 20,000 vertex roots are more than the wavefronts launched
    assert lds_dev // 5 < one.lds <= lds_dev and all(r.lds <= one.lds for r in rs)
    if d.d_max <= 128:
        assert one.lds <= lds_dev // 2 and min(r.lds for r in rs) < one.lds
    for r in rs:   # admitted before its start and until its end
        assert sum(x.lds for x in rs if x.t_start <= r.t_start < x.t_done) <= lds_dev
