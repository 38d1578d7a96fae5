"""Degree orientation at the edges of its kernels' tiles, row by row against NumPy, and
the symmetry check on graphs with as many entries missing upwards as downwards."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def hubs(n, sizes, seed):
    """A sparse background with hubs of the given degrees, joined to one another."""
    rng = np.random.default_rng(seed)
    e = [np.stack([rng.integers(0, n, 2 * n), rng.integers(0, n, 2 * n)], 1)]
    for h, s in enumerate(sizes):
        leaf = rng.permutation(n)[:s]
        e.append(np.stack([np.full(leaf.size, h), leaf], 1))
    i, j = np.triu_indices(len(sizes), 1)
    e.append(np.stack([i, j], 1))
    return synth.from_pairs(n, np.concatenate(e))


GRAPHS = [  # 2048 and 8192: scan and sort tiles; 256 / 64: rows handled by 16 lanes; 1024: rows sorted in LDS
    lambda: synth.complete(65), lambda: synth.complete(66), lambda: synth.complete(257), lambda: synth.complete(1026),
    lambda: hubs(2048, [255, 256, 257, 2000], 1), lambda: hubs(2049, [64, 65, 66], 2),
    lambda: hubs(8192, [300] * 70, 3), lambda: hubs(8193, [4000, 5000], 4), lambda: hubs(70001, [1025, 60000], 5),
]


@pytest.mark.parametrize("i", range(len(GRAPHS)))
def test_degree_orientation_rows(kc, i):
    g = GRAPHS[i]()
    d = kc.orient(kc.to_device(g), kc.ORDER_DEGREE)
    rp, col, src, perm = kc.dag_to_host(d)
    deg = g.degrees()
    want = np.lexsort((np.arange(g.n), deg))
    assert np.array_equal(perm, want)
    rank = np.empty(g.n, np.int64)
    rank[want] = np.arange(g.n)
    a, b = rank[np.repeat(np.arange(g.n), deg)], rank[g.col]
    key = np.sort((a * g.n + b)[a < b])
    assert np.array_equal(src, key // g.n) and np.array_equal(col, key % g.n)
    out = np.bincount(key // g.n, minlength=g.n)
    assert np.array_equal(rp, np.concatenate([[0], np.cumsum(out)]))
    assert d.d_max == out.max()


@pytest.mark.parametrize("hub", [40, 3000])
def test_missing_reverse_entries_are_found_in_both_directions(kc, hub):
    import torch
    g = hubs(5000, [hub], 6)
    deg = g.degrees()
    row = np.repeat(np.arange(g.n), deg)
    down = (deg[g.col] < deg[row]) & (row < 100)
    up = (deg[g.col] > deg[row]) & (row >= 100)
    down, up = np.nonzero(down)[0], np.nonzero(up)[0]
    for drop in (down[:2], up[-2:], [down[0], up[-1]]):
        keep = np.ones(g.nnz, bool)
        keep[drop] = False
        rp = np.concatenate([[0], np.cumsum(np.bincount(row[keep], minlength=g.n))]).astype(np.int32)
        bad = kc.Csr(g.n, torch.as_tensor(rp).cuda(), torch.as_tensor(g.col[keep]).cuda())
        for order in (kc.ORDER_DEGREE, kc.ORDER_DEGENERACY, kc.ORDER_COLOR):
            with pytest.raises(kc.KcError) as e:
                kc.orient(bad, order)
            assert e.value.code == kc.EINVAL


@pytest.mark.parametrize("h", [1, 2, 3, 4, 5, 8, 16, 31, 32, 33, 127, 128, 129])
def test_one_wrong_entry_is_found_at_any_place_of_a_row(kc, h):
    # rows of 2h entries of one length (256: rows of a wavefront, longer: of the block); the
    # wrong entry keeps the row sorted, and as many entries as before point up and down
    import torch
    n = 4 * h + 301
    off = np.concatenate([-2 * np.arange(h, 0, -1), 2 * np.arange(1, h + 1)])
    col = np.sort((np.arange(n)[:, None] + off[None, :]) % n, axis=1).astype(np.int32)
    rp = torch.as_tensor(np.arange(n + 1, dtype=np.int32) * 2 * h).cuda()
    assert kc.orient(kc.Csr(n, rp, torch.as_tensor(col.reshape(-1)).cuda()), kc.ORDER_DEGREE).m == n * h
    for v in (2 * h, 2 * h + 77, n - 2 * h - 2):
        for at in sorted({0, h // 2, h - 1, h, h + h // 2, 2 * h - 1}):
            wrong = col.copy()
            wrong[v, at] += 1
            bad = kc.Csr(n, rp, torch.as_tensor(wrong.reshape(-1)).cuda())
            with pytest.raises(kc.KcError) as e:
                kc.orient(bad, kc.ORDER_DEGREE)
            assert e.value.code == kc.EINVAL, (v, at)
