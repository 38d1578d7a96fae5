"""Degeneracy orientation while another stream's count holds every compute unit: the peel's
workgroups do not fit beside it, and the call waits until the count has ended."""
import threading
import time

import pytest

import synth
from test_gpu_cancel import HostFlag

pytestmark = pytest.mark.gpu

HOLD = 12.0   # seconds: more than a barrier wait of the peel lasts


def test_orient_waits_for_a_long_count(kc):
    import torch
    g = kc.to_device(synth.chung_lu(20011, 2.1, 16.0, 800.0, 3))
    want = kc.orient(g, kc.ORDER_DEGENERACY)
    # 13-cliques among 700 vertices at density 0.6: hours, 76 KB of LDS for each wavefront
    hog = kc.orient(kc.to_device(synth.erdos_renyi(700, 0.6, 1)), kc.ORDER_DEGENERACY)
    torch.cuda.synchronize()
    flag, status, got, took = HostFlag(), [], [], []

    def count():
        with torch.cuda.stream(torch.cuda.Stream()):
            status.append(kc.count_status(hog, 13, scheme=kc.SCHEME_VC, cancel=flag.addr)[0])

    def orient():
        t0 = time.monotonic()
        with torch.cuda.stream(torch.cuda.Stream()):
            got.append(kc.orient(g, kc.ORDER_DEGENERACY))
        took.append(time.monotonic() - t0)

    threads = [threading.Thread(target=count), threading.Thread(target=orient)]
    threads[0].start()
    time.sleep(0.5)
    threads[1].start()
    time.sleep(HOLD)
    still_running = not status
    flag.set(1)
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    flag.free()
    assert still_running and status == [kc.ECANCELED]
    print("orientation took %.2f s of %.1f" % (took[0], HOLD))
    assert (got[0].d_max, got[0].degeneracy) == (want.d_max, want.degeneracy)
    for a, b in ((got[0].row_ptr, want.row_ptr), (got[0].col, want.col), (got[0].perm, want.perm)):
        assert torch.equal(a, b)
