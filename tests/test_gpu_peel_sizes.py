"""Degeneracy order where the peel's work is split: one workgroup does all rounds up to 4,000
vertices, and a block of the whole-device rounds gathers at most 16,384 vertices a round."""
import numpy as np
import pytest

import synth
from test_gpu_peel import peel, star_core

pytestmark = pytest.mark.gpu

SMALL = [f for n in (3999, 4000, 4001)
         for f in (lambda n=n: synth.erdos_renyi(n, 0.002, n), lambda n=n: star_core(n, 600, n))]


@pytest.mark.parametrize("i", range(len(SMALL)))
def test_one_workgroup_or_the_device(kc, i):
    g = SMALL[i]()
    rnd, degen = peel(g)
    d = kc.orient(kc.to_device(g), kc.ORDER_DEGENERACY)
    assert d.degeneracy == degen
    assert np.array_equal(kc.dag_to_host(d)[3], np.lexsort((np.arange(g.n), rnd)))


# 16 blocks for 278,528 vertices (17,408 each), 64 for 1,048,576 + 64,000
@pytest.mark.parametrize("n", [278_528, 1_112_576])
@pytest.mark.parametrize("kind", ["empty", "matching", "cycle"])
def test_frontier_beyond_the_blocks_buffers(kc, kind, n):
    if kind == "empty":
        g = synth.empty(n)
    elif kind == "matching":
        g = synth.from_pairs(n, np.arange(n).reshape(-1, 2))
    else:
        g = synth.cycle(n)
    d = kc.orient(kc.to_device(g), kc.ORDER_DEGENERACY)
    assert d.degeneracy == {"empty": 0, "matching": 1, "cycle": 2}[kind]
    assert np.array_equal(kc.dag_to_host(d)[3], np.arange(n))       # one round takes all
