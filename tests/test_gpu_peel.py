"""Degeneracy order against a plain level-synchronous peel, vertex by vertex.

The order is (round, id): rounds are fixed by the peeling rule alone, so the whole
permutation must agree, on both sides of the size (26,000 vertices) from which the
whole-device rounds may leave the last ones to one workgroup.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def peel(g):
    """(round of every vertex, degeneracy)."""
    rp, col = g.row_ptr.astype(np.int64), g.col
    deg = np.diff(rp)
    rnd = np.full(g.n, -1)
    r, c = 0, -1
    front = np.zeros(0, np.int64)
    while (rnd < 0).any():
        if front.size == 0:
            c = int(deg[rnd < 0].min())
            front = np.nonzero((rnd < 0) & (deg <= c))[0]
        rnd[front] = r
        r += 1
        nb = np.concatenate([col[rp[v]:rp[v + 1]] for v in front]) if front.size else col[:0]
        before = deg.copy()
        np.subtract.at(deg, nb, 1)
        front = np.nonzero((rnd < 0) & (before > c) & (deg <= c))[0]
    return rnd, max(c, 0)


def star_core(n, core, seed):
    """A clique whose members also have a long row of leaves each (rows far beyond a
    wavefront), over a sparse background."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(core, 1)
    hub = np.repeat(np.arange(4), 3 * core)
    leaf = rng.integers(core, n, hub.size)
    a, b = rng.integers(core, n, 2 * n), rng.integers(core, n, 2 * n)
    return synth.from_pairs(n, np.concatenate([np.stack([i, j], 1), np.stack([hub, leaf], 1), np.stack([a, b], 1)]))


GRAPHS = [
    lambda: synth.empty(1), lambda: synth.complete(2), lambda: synth.complete(70), lambda: synth.empty(26001),
    lambda: synth.erdos_renyi(1025, 0.02, 5), lambda: synth.erdos_renyi(25999, 0.0003, 6),
    lambda: synth.erdos_renyi(26001, 0.0004, 7), lambda: star_core(26000, 300, 8), lambda: star_core(60013, 700, 9),
    lambda: synth.chung_lu(70001, 2.1, 12.0, 1500.0, 10),
]


@pytest.mark.parametrize("i", range(len(GRAPHS)))
def test_degeneracy_order_is_the_peeling_order(kc, i):
    g = GRAPHS[i]()
    rnd, degen = peel(g)
    d = kc.orient(kc.to_device(g), kc.ORDER_DEGENERACY)
    perm = kc.dag_to_host(d)[3]
    assert d.degeneracy == degen
    assert np.array_equal(perm, np.lexsort((np.arange(g.n), rnd)))
