"""Pivot totals at the candidate-set sizes where the walk changes (64: one word pair in
registers, 128: two, beyond: rows in LDS), against the oracle, with frames handed over as
early as the thresholds allow and with none."""
import math

import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def dense(n, p, seed):
    """G(n, p) joined to one vertex per side, so that some root has n candidates."""
    return synth.join(synth.erdos_renyi(n, p, seed), synth.empty(1))


CASES = [(n, p) for n in (31, 33, 63, 64, 65, 66) for p in (0.5, 0.9)] + [(n, 0.5) for n in (127, 128, 129, 130)]


@pytest.mark.parametrize("n,p", CASES)
def test_totals_at_the_word_boundaries(kc, n, p):
    g = dense(n, p, n)
    want, om = oracle.count_all(oracle.orient(g, oracle.DEGENERACY), True, oracle.VC)
    for order in (kc.ORDER_DEGREE, kc.ORDER_DEGENERACY):
        d = kc.orient(kc.to_device(g), order)
        for scheme in (kc.SCHEME_VC, kc.SCHEME_EC):
            for handoff, after in ((False, 0), (True, 1)):
                st, got, gom = kc.count_all_status(d, True, scheme=scheme, handoff=handoff, handoff_after=after,
                                                   handoff_every=after)
                assert (st, gom) == (kc.OK, om)
                assert got[:om + 1] == want[:om + 1] and not any(got[om + 1:])
                for k in (3, 4, om // 2 + 1, om - 1, om, om + 1):
                    if k >= 3:
                        assert kc.count(d, k, pivot=True, scheme=scheme, handoff=handoff, handoff_after=after,
                                        handoff_every=after) == (want[k] if k <= om else 0), k


@pytest.mark.parametrize("n", [65, 66, 129, 130])
def test_cliques_and_their_complements(kc, n):
    # every vertex is adjacent to all others (a clique), or to all but one (a cocktail party)
    d = kc.orient(kc.to_device(synth.complete(n)), kc.ORDER_DEGREE)
    got, om = kc.count_all(d)
    assert om == n and got[:n + 1] == [math.comb(n, j) for j in range(n + 1)]
    pairs = 20
    d = kc.orient(kc.to_device(synth.join(synth.complete(n - 2 * pairs), synth.complete_multipartite([2] * pairs))),
                  kc.ORDER_DEGREE)
    want = [sum(math.comb(n - 2 * pairs, j - i) * math.comb(pairs, i) * 2 ** i for i in range(min(j, pairs) + 1))
            for j in range(n - pairs + 1)]
    got, om = kc.count_all(d)
    assert om == n - pairs and got[:om + 1] == want
