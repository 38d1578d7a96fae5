"""Graphs without reverse entries, given with validate=False: the DAG is unspecified and the
call may refuse it, but every access stays in the caller's arrays."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GUARD = 4096


def directed(kc, n, edges):
    """The CSR with exactly these directed edges."""
    import torch
    e = np.unique(edges[:, 0].astype(np.int64) * n + edges[:, 1])
    rp = np.concatenate([[0], np.cumsum(np.bincount(e // n, minlength=n))]).astype(np.int32)
    return kc.Csr(n, torch.as_tensor(rp).cuda(), torch.as_tensor((e % n).astype(np.int32)).cuda())


def both(a, b):
    return np.concatenate([np.stack([a, b], 1), np.stack([b, a], 1)])


def orient_guarded(kc, g, order):
    """Status of the call; arrays and workspace (full of stale words) must end as they began."""
    import torch
    m = g.nnz // 2

    def guarded(count):
        return torch.full((count + GUARD,), -7, dtype=torch.int32, device="cuda")

    out = kc.Dag(g.n, m, 0, -1, order, guarded(g.n + 1), guarded(m), guarded(m), guarded(g.n))
    need = kc.orient_workspace_bytes(g.n, g.nnz, order)
    ws = torch.full((need + GUARD,), 255, dtype=torch.uint8, device="cuda")
    status = kc.OK
    try:
        kc.orient(g, order, validate=False, ws=ws[:need], out=out)
    except kc.KcError as e:
        status = e.code
    torch.cuda.synchronize()
    for t, count in ((out.row_ptr, g.n + 1), (out.col, m), (out.src, m), (out.perm, g.n)):
        assert bool((t[count:] == -7).all())
    assert bool((ws[need:] == 255).all())
    return status


@pytest.mark.parametrize("fan", [63, 64, 65, 66, 300, 1500])
def test_peel_with_neighbours_that_left_without_a_reverse_entry(kc, fan):
    # 1500 vertices without entries leave first, a path of 3000 takes 1500 rounds (so that the
    # whole-device rounds end early), and 100 vertices list `fan` of the first 1500
    rng = np.random.default_rng(fan)
    path = np.arange(1500, 4499)
    hub = np.arange(4500, 4600)
    one_way = np.concatenate([np.stack([np.full(fan, h), rng.permutation(1500)[:fan]], 1) for h in hub])
    e = np.concatenate([both(path, path + 1), one_way])
    g = directed(kc, 4600, e)
    assert orient_guarded(kc, g, kc.ORDER_DEGENERACY) == kc.EINVAL


@pytest.mark.parametrize("order", [0, 1, 3])
@pytest.mark.parametrize("fan", [20, 200, 1300])
def test_more_entries_kept_than_the_arrays_hold(kc, order, fan):
    # 1000 vertices list `fan` of 1400 that list only one another: almost every entry points
    # to the later end of its edge, twice as many as m
    rng = np.random.default_rng(fan)
    i, j = np.triu_indices(1400, 1)
    near = (j - i) <= fan                          # rows of the 1400 longer than `fan`
    one_way = np.concatenate([np.stack([np.full(fan, 1400 + v), rng.permutation(1400)[:fan]], 1) for v in range(1000)])
    g = directed(kc, 2400, np.concatenate([both(i[near], j[near]), one_way]))
    status = orient_guarded(kc, g, order)
    if order == kc.ORDER_DEGREE:
        assert status == kc.EINVAL


@pytest.mark.parametrize("fan", [20, 200])
def test_approximate_rounds_end_when_none_can_leave(kc, fan):
    # the 1400 lose `fan` degrees to each of 1000 vertices that they do not list: their degrees
    # sum to less than zero, and none is at most 1.1 times that average
    rng = np.random.default_rng(fan)
    i, j = np.triu_indices(1400, 1)
    near = (j - i) <= fan
    one_way = np.concatenate([np.stack([np.full(fan, 1400 + v), rng.permutation(1400)[:fan]], 1) for v in range(1000)])
    g = directed(kc, 2400, np.concatenate([both(i[near], j[near]), one_way]))
    assert orient_guarded(kc, g, kc.ORDER_APPROX_DEGENERACY) == kc.EINVAL
