"""Graphs without an arc below 0.9 run their rounds by word (whose reverse tasks start on the first engine
tier), one arc below that brings the rounds by snapshot back; single calls, plans, lazy calls and batches, against
the oracle."""
import numpy as np
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


def _graph(n, m, seed, low):
    """Probabilities from 0.9 on, and one of `low` if it is not None."""
    g = gg.chung_lu_graph(n, m, 2.5, seed, True, 1.0)
    p = np.random.default_rng(seed).choice(np.array([0.9, 0.95, 1.0], np.float32), g.m)
    if low is not None:
        p[g.m // 2] = low
    return gg.Graph(g.n, g.row_ptr, g.col, p.astype(np.float32))


def _lists(pair):
    return [x.cpu().tolist() for x in pair]


@pytest.mark.parametrize("low,by_word", [(None, True), (0.9, True), (np.nextafter(np.float32(0.9), np.float32(0)), False),
                                         (0.0, False)])
def test_rounds_of_sure_arcs(im, low, by_word):
    import torch
    g = _graph(1200, 5000, 71, low)
    h = _graph(300, 900, 72, None)
    R, k = 70, 6
    s_ref, g_ref, tr_ref, _ = oracle.select_du(g.row_ptr, g.col, g.prob, R, k, 4, trace=True)
    ref = [s_ref.tolist(), g_ref.tolist()]
    href = [x.tolist() for x in oracle.select_du(h.row_ptr, h.col, h.prob, 130, 3, 5)[:2]]
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    dh = im.Graph.from_numpy(h.row_ptr, h.col, h.prob, device="cuda:0")
    ws = im.Workspace()
    seeds, gains, tr = im.select(d, R, k, 4, ws=ws, trace=True)
    assert _lists((seeds, gains)) == ref
    assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
    assert (ws.stats()["reached_rev_t0"] > 0) == by_word
    assert _lists(im.select_lazy(d, R, k, 4, ws=ws)) == ref
    out = [_lists(x) for x in im.select_batch([(d, R, k, 4), (dh, 130, 3, 5)], ws=ws)]
    assert out == [ref, href]
    assert (ws.stats()["reached_rev_t0"] > 0) == by_word
    plan = im.Plan(d, R, k, 4)
    for _ in range(3):
        plan.launch()
        torch.cuda.synchronize()
        assert _lists((plan.seeds, plan.gains)) == ref
        im.select(dh, 130, 3, 5, ws=ws)   # eager work between the replays
    plan.close()


@pytest.mark.parametrize("m,by_word", [(2399, False), (2400, True)])
def test_thin_graphs_stay_by_snapshot(im, m, by_word):
    g = _graph(1200, m, 73, None)
    s_ref, g_ref, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, 65, 5, 4)
    ws = im.Workspace()
    seeds, gains, _ = im.select(im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0"), 65, 5, 4, ws=ws)
    assert _lists((seeds, gains)) == [s_ref.tolist(), g_ref.tolist()]
    assert (ws.stats()["reached_rev_t0"] > 0) == by_word
