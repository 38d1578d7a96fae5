"""Orientation in a workspace that is aligned to words only, as one carved out of a larger
buffer may be."""
import pytest

import synth

pytestmark = pytest.mark.gpu

GRAPHS = [lambda: synth.complete(70), lambda: synth.erdos_renyi(4000, 0.01, 1),
          lambda: synth.chung_lu(70001, 2.1, 12.0, 1500.0, 10)]


@pytest.mark.parametrize("words", [1, 3])
@pytest.mark.parametrize("i", range(len(GRAPHS)))
def test_workspace_aligned_to_words(kc, i, words):
    import torch
    g = kc.to_device(GRAPHS[i]())
    for order in (kc.ORDER_DEGREE, kc.ORDER_DEGENERACY, kc.ORDER_COLOR):
        need = kc.orient_workspace_bytes(g.n, g.nnz, order)
        ws = torch.empty(need + 64, dtype=torch.uint8, device="cuda")[4 * words:4 * words + need]
        assert ws.data_ptr() % 8 == 4
        a, b = kc.orient(g, order), kc.orient(g, order, ws=ws)
        assert (a.d_max, a.degeneracy) == (b.d_max, b.degeneracy)
        for x, y in ((a.row_ptr, b.row_ptr), (a.col, b.col), (a.src, b.src), (a.perm, b.perm)):
            assert torch.equal(x, y)
