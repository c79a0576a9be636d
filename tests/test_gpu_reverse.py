"""Reverse searches of up to 64 sources of one snapshot: sizes around a task's 64 sources and around
the limits of its two LDS tables (past the larger one it runs in global memory), against the oracle."""
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


def _graph(n, arcs, p):
    src, dst = (np.array(a, np.int64) for a in zip(*arcs))
    row_ptr, col = gg.to_csr(n, src, dst)
    return gg.Graph(n, row_ptr, col, gg.uniform_prob(len(col), p))


def _fan(sinks, p):
    """Node 0 reaches every sink (one task per 64 of them and snapshot); every sink has two
    more in-arcs, one of them from a node that reaches all."""
    n = 2 * sinks + 2
    arcs = [(0, 2 + i) for i in range(sinks)] + [(1, 2 + i) for i in range(sinks)]
    return _graph(n, arcs + [(2 + sinks + i, 2 + i) for i in range(sinks)], p)


def _in_star(leaves, p):
    """A search from the centre visits the leaves and itself."""
    return _graph(leaves + 3, [(i, leaves) for i in range(leaves)] +
                  [(leaves, leaves + 1), (leaves + 1, leaves + 2)], p)


CASES = [("fan", s, p) for s in (1, 63, 64, 65, 129) for p in (0.5, 1.0)]
CASES += [("star", n, 1.0) for n in (1638, 1639, 1640, 3198, 3199, 3200, 5000)]


@pytest.mark.parametrize("kind,size,p", CASES, ids=lambda v: str(v))
@pytest.mark.parametrize("hub", [0, 256])
def test_reverse_search_sizes(im, kind, size, p, hub):
    g = _fan(size, p) if kind == "fan" else _in_star(size, p)
    R, k, seed = 66, 3, 11
    s_ref, g_ref, tr_ref, st = oracle.select_du(g.row_ptr, g.col, g.prob, R, k, seed, trace=True)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    ws.set_hub_degree(hub)   # 0: the star's centre is expanded through its masks
    seeds, gains, tr = im.select(d, R, k, seed, ws=ws, trace=True)
    assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
    assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
    gs = ws.stats()
    assert gs["trav_rev"] == st["trav_rev"] and gs["decrements"] == st["decrements"]


def test_reverse_search_batch_bins(im):
    """A batch's sources are grouped by instance: uneven instances, ragged R and no arcs at all."""
    insts = [(_fan(70, 0.4), 65, 3, 5), (_in_star(3300, 1.0), 2, 2, 6), (_fan(3, 0.9), 130, 2, 7),
             (_in_star(1700, 1.0), 64, 3, 8)]
    dev = [(im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0"), R, k, s)
           for g, R, k, s in insts]
    for (g, R, k, s), (seeds, gains) in zip(insts, im.select_batch(dev)):
        s_ref, g_ref, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, R, k, s)
        assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
