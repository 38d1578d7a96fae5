"""Batches whose max_degree is below a hub's degree: it sizes the sort, so the order may
change, but every clique is counted and credited to its own graph."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def pack(kc, graphs):
    voff = np.concatenate([[0], np.cumsum([g.n for g in graphs])]).astype(np.int32)
    at = np.concatenate([[0], np.cumsum([g.nnz for g in graphs])])
    rp = np.concatenate([[0]] + [g.row_ptr[1:].astype(np.int64) + a for g, a in zip(graphs, at)]).astype(np.int32)
    col = np.concatenate([g.col + v for g, v in zip(graphs, voff)]).astype(np.int32)
    return kc.batch_to_device(synth.Batch(voff, rp, col))


def wheel(n, seed):
    """A hub joined to all of a sparse graph: one long row, short out-rows in any order but the
    hub's own, which stays under 32 candidates for n <= 33."""
    return synth.join(synth.erdos_renyi(n - 1, 4.0 / n, seed), synth.empty(1))


@pytest.mark.parametrize("graphs", [1, 2, 40, 300])
@pytest.mark.parametrize("bound", [0, 1, 3, 8, 20])
def test_counts_do_not_depend_on_the_bound(kc, graphs, bound):
    gs = [wheel(20 + i % 13, i) for i in range(graphs)]
    bd = dataclasses.replace(pack(kc, gs), max_degree=bound, max_graph_edges=0)
    for k in (3, 4):
        want = [oracle.count(oracle.orient(g, oracle.DEGREE), k) for g in gs]
        assert kc.batch_count(bd, k) == want
        assert kc.batch_count(bd, k, kc.BatchPlan.make([(1 << 30, kc.SCHEME_EC)])) == want
