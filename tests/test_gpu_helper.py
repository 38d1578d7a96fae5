"""The helper launch of a deep count: roots that the main launch has claimed are not walked
again, whether subtrees are handed over or not, and with more roots than two per wavefront."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("left", [200, 20000])
def test_every_root_is_walked_once(kc, left):
    # Each of `left` vertices has the same 40 neighbours, none of them adjacent: a root's 40
    # candidates hold no edge, so it has no pair task that another wavefront could join for, and
    # takes as many rounds of its wavefront whoever else runs.
    pairs = np.stack([np.repeat(40 + np.arange(left), 40), np.tile(np.arange(40), left)], 1)
    d = kc.orient(kc.to_device(synth.from_pairs(40 + left, pairs)), kc.ORDER_DEGENERACY)
    assert d.d_max == 40
    rounds = {}
    for handoff in (True, False):
        for single in (True, False):
            p = kc.Profile()
            assert kc.count(d, 7, scheme=kc.SCHEME_VC, profile=p, collect_stats=True, handoff=handoff,
                            single_stream=single) == 0
            assert p.roots_width[1] == left
            rounds[handoff, single] = p.iters_width[1]
    assert min(rounds.values()) >= left
    assert len(set(rounds.values())) == 1, rounds
