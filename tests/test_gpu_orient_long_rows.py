"""Orientation of rows beyond 256 entries, at the edges of who handles them: a wavefront up to
2048 entries of which at most 316 are kept, the block otherwise; one row or four per wavefront."""
import numpy as np
import pytest

import synth
from test_gpu_orient_edges import hubs

pytestmark = pytest.mark.gpu


def clique_and_leaves(core, leaves, n, seed):
    """A clique whose members keep up to core - 1 neighbours of rows of core - 1 + leaves."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(core, 1)
    leaf = np.concatenate([core + rng.permutation(n - core)[:leaves] for _ in range(core)])
    return synth.from_pairs(n, np.concatenate([np.stack([i, j], 1),
                                               np.stack([np.repeat(np.arange(core), leaves), leaf], 1)]))


GRAPHS = [
    lambda: synth.complete(258), lambda: synth.complete(317), lambda: synth.complete(318), lambda: synth.complete(321),
    lambda: synth.erdos_renyi(1500, 0.4, 1), lambda: synth.erdos_renyi(3001, 0.17, 2),
    lambda: hubs(9000, [2047, 2048, 2049, 2050], 3), lambda: hubs(30011, [257] * 40 + [2048] * 20 + [2500] * 3, 4),
    lambda: clique_and_leaves(317, 1700, 4000, 5), lambda: clique_and_leaves(318, 1740, 4000, 6),
    lambda: clique_and_leaves(300, 1749, 70001, 7),
]


@pytest.mark.parametrize("order", [0, 1])
@pytest.mark.parametrize("i", range(len(GRAPHS)))
def test_rows(kc, i, order):
    g = GRAPHS[i]()
    d = kc.orient(kc.to_device(g), order)
    rp, col, src, perm = kc.dag_to_host(d)
    deg = g.degrees()
    if order == kc.ORDER_DEGREE:
        assert np.array_equal(perm, np.lexsort((np.arange(g.n), deg)))
    rank = np.empty(g.n, np.int64)
    rank[perm] = np.arange(g.n)
    a, b = rank[np.repeat(np.arange(g.n), deg)], rank[g.col]
    key = np.sort((a * g.n + b)[a < b])
    assert np.array_equal(src, key // g.n) and np.array_equal(col, key % g.n)
    out = np.bincount(key // g.n, minlength=g.n)
    assert np.array_equal(rp, np.concatenate([[0], np.cumsum(out)])) and d.d_max == out.max()
