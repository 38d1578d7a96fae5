"""The width lists of a count's roots: sizes at every list's border, and root counts at the
edges of the blocks' shares (1,024 roots a block, 512 blocks), in closed form."""
import math

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def cliques(n, sizes, edges=0):
    """Disjoint cliques and single edges at the given places, scattered over n vertices."""
    at = np.random.default_rng(n).permutation(n)
    pairs, used = [], 0
    for c in sizes:
        i, j = np.triu_indices(c, 1)
        pairs.append(np.stack([at[used + i], at[used + j]], 1))
        used += c
    pairs.append(at[used:used + 2 * edges].reshape(-1, 2))
    return synth.from_pairs(n, np.concatenate(pairs))


BORDERS = [33, 34, 65, 66, 129, 130, 257, 258]


# a clique of c vertices has vertex roots of 0 .. c - 1 candidates
@pytest.mark.parametrize("n", [514, 1023, 1024, 1025, 2049, 524287, 524288, 524289, 526337])
def test_vertex_roots(kc, n):
    sizes = [514] if n < 2000 else BORDERS + [513, 514]
    if n == 2049:
        sizes = BORDERS + [514]
    d = kc.orient(kc.to_device(cliques(n, sizes)), kc.ORDER_DEGREE)
    for k in (3, 4):
        assert kc.count(d, k, scheme=kc.SCHEME_VC) == sum(math.comb(c, k) for c in sizes), k


@pytest.mark.parametrize("m", [1023, 1024, 1025, 2049, 524287, 524288, 524289, 525313])
def test_edge_roots(kc, m):
    sizes = [34, 32] if m < 5000 else BORDERS + [514, 300]
    edges = m - sum(math.comb(c, 2) for c in sizes)
    if edges < 0:
        sizes, edges = [33], m - math.comb(33, 2)
    d = kc.orient(kc.to_device(cliques(sum(sizes) + 2 * edges + 1, sizes, edges)), kc.ORDER_DEGREE)
    assert d.m == m
    for k in (3, 4, 5):
        assert kc.count(d, k, scheme=kc.SCHEME_EC) == sum(math.comb(c, k) for c in sizes), k


def test_batch_of_cliques(kc):
    # graphs of one, two and more shares, and empty ones between them
    gs = [synth.complete(33), synth.empty(1024), cliques(1025, [65, 66, 129]), synth.empty(1), synth.complete(258)]
    voff = np.concatenate([[0], np.cumsum([g.n for g in gs])])
    eoff = np.concatenate([[0], np.cumsum([g.col.size for g in gs])])
    row_ptr = np.concatenate([g.row_ptr[:-1].astype(np.int64) + e for g, e in zip(gs, eoff)] + [eoff[-1:]])
    b = synth.Batch(voff.astype(np.int32), row_ptr.astype(np.int32),
                    np.concatenate([g.col + v for g, v in zip(gs, voff)]).astype(np.int32))
    for plan in (None, kc.BatchPlan.make([(1 << 30, kc.SCHEME_EC)]), kc.BatchPlan.make([(1 << 30, kc.SCHEME_VC)])):
        for k in (3, 4):
            want = [math.comb(33, k), 0, sum(math.comb(c, k) for c in (65, 66, 129)), 0, math.comb(258, k)]
            assert kc.batch_count(kc.batch_to_device(b), k, plan) == want, k


@pytest.mark.parametrize("n", [514, 1025, 2049, 524289])
def test_local_counts_and_lists(kc, n):
    # d_max 513 would not fit a wavefront's LDS: sizes up to 258
    sizes = [258] if n == 514 else BORDERS
    g = cliques(n, sizes)
    d = kc.orient(kc.to_device(g), kc.ORDER_DEGREE)
    deg = g.degrees()
    for scheme in (kc.SCHEME_VC, kc.SCHEME_EC):
        for k in (3, 4):
            want = [math.comb(x, k - 1) for x in range(258)]
            got = kc.count_local(d, k, scheme=scheme).cpu().numpy()
            assert np.array_equal(got, np.array(want)[deg]), k
        total, rows = kc.list_cliques(d, 3, scheme=scheme)
        rows = np.sort(rows.cpu().numpy().astype(np.int64), axis=1)
        assert total == rows.shape[0] == sum(math.comb(c, 3) for c in sizes)
        assert np.unique((rows[:, 0] * n + rows[:, 1]) * n + rows[:, 2]).size == total
