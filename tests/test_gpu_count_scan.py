"""Initial counts of a hub whose live lists do not fit (most of its arcs live in many snapshots): around
the arcs that one wavefront still reads by mask, on bitmaps and on tables, alone, behind a few nodes and
behind thousands; gains and the traversal counter against the oracle."""
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


def _graph(n, arcs, p, back):
    """Node 0 has `arcs` arcs of probability p; `back` nodes lead to it."""
    src = np.concatenate([np.zeros(arcs, np.int64), np.arange(1, back + 1)])
    dst = np.concatenate([np.arange(1, arcs + 1), np.zeros(back, np.int64)])
    pr = np.concatenate([np.full(arcs, p), np.full(back, 0.3)])
    row_ptr = np.zeros(n + 1, np.uint64)
    row_ptr[1:] = np.cumsum(np.bincount(src, minlength=n))
    return gg.Graph(n, row_ptr, dst.astype(np.uint32), pr.astype(np.float32))


@pytest.mark.parametrize("n,arcs,p,back,R", [
    (18000, 16383, 0.5, 0, 65), (18000, 16384, 0.5, 3, 65), (18000, 16385, 0.5, 3, 65), (40000, 30000, 0.3, 40, 130),
    (60000, 30000, 0.2, 3000, 20), (260000, 16384, 0.05, 5, 70), (260000, 16385, 0.05, 5, 70), (260000, 100000, 0.5, 4, 64)])
def test_hub_without_lists(im, n, arcs, p, back, R):
    g = _graph(n, arcs, p, back)
    ref, st = oracle.initial_gains(g.row_ptr, g.col, g.prob, R, 5)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):   # the second call finds the shared marks as the first left them
        got = im.initial_gains(d, R, 5, ws=ws).cpu().numpy()
        assert np.array_equal(got, ref.astype(np.int64))
        assert ws.stats()["trav_init"] == st["trav_init"]
