"""An update strategy of single graphs leaves batches and lazy calls on the rounds by snapshot."""
import pytest

import oracle
from paper_1212_4779_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def im():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4779_amd as im
    return im


def _dev(im, g):
    return im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")


def test_update_strategy_leaves_batches_alone(im):
    insts, refs = [], []
    for i in range(3):
        g = gg.chung_lu_graph(500 + 300 * i, 4000, 2.5, 90 + i, True, None if i % 2 else 0.08)
        insts.append((_dev(im, g), 100, 5, 3 + i))
        s, gn, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, 100, 5, 3 + i)
        refs.append([s.tolist(), gn.tolist()])
    ws = im.Workspace()
    ws.set_affected_gain(1 << 62)
    out = [[s.cpu().tolist(), gn.cpu().tolist()] for s, gn in im.select_batch(insts, ws=ws)]
    assert out == refs
    assert ws.stats()["reached_rev_t0"] == 0   # by snapshot: no task starts on the first tier
    (d, R, k, seed), ref = insts[0], refs[0]
    seeds, gains, _ = im.select(d, R, k, seed, ws=ws)
    assert [seeds.cpu().tolist(), gains.cpu().tolist()] == ref and ws.stats()["trav_rev"] == 0
    seeds, gains = im.select_lazy(d, R, k, seed, ws=ws)
    assert [seeds.cpu().tolist(), gains.cpu().tolist()] == ref
