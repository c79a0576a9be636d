"""The largest initial-count tasks, one snapshot per wavefront: instances around the sizes where the
visited sets change (bitmaps of eight and of four wavefronts, tables), searches around the table's
limit, snapshots that share their nodes (handed to the dense tier), and the queue's part in LDS;
gains and word counters against the oracle."""
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


def _graph(n, leaves, p, tail):
    """A hub with arcs of probability p to the leaves, every tenth of which starts a path of
    `tail` nodes (p = 0.8), some of them back to the hub."""
    src, dst, pr = [np.zeros(leaves, np.int64)], [np.arange(1, leaves + 1)], [np.full(leaves, p)]
    first = leaves + 1
    for i in range(0, leaves, 10):
        nodes = np.concatenate([[1 + i], first + np.arange(tail)])
        first += tail
        src.append(nodes[:-1])
        dst.append(nodes[1:])
        pr.append(np.full(tail, 0.8))
        if i % 100 == 0:
            src.append(nodes[-1:])
            dst.append(np.zeros(1, np.int64))
            pr.append(np.full(1, 0.5))
    assert first <= n
    src, dst, pr = np.concatenate(src), np.concatenate(dst), np.concatenate(pr)
    order = np.lexsort((dst, src))
    row_ptr = np.zeros(n + 1, np.uint64)
    row_ptr[1:] = np.cumsum(np.bincount(src, minlength=n))
    return gg.Graph(n, row_ptr, dst[order].astype(np.uint32), pr[order].astype(np.float32))


@pytest.mark.parametrize("n,leaves,p,tail,R", [
    (5000, 2000, 0.1, 3, 130), (5000, 2000, 0.9, 3, 70), (131072, 1200, 0.2, 5, 65),
    (131073, 1200, 0.2, 5, 65), (235904, 1200, 0.2, 5, 65), (235936, 1200, 0.2, 5, 65),
    (236000, 2900, 0.9, 2, 3), (236000, 3400, 0.9, 2, 3), (236000, 6200, 0.4, 2, 66),
    (236000, 3000, 1.0, 2, 64),
])
def test_counts_by_snapshot(im, n, leaves, p, tail, R):
    g = _graph(n, leaves, p, tail)
    ref, st = oracle.initial_gains(g.row_ptr, g.col, g.prob, R, 5)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):   # the second call finds the shared bitmaps as the first left them
        got = im.initial_gains(d, R, 5, ws=ws).cpu().numpy()
        assert np.array_equal(got, ref.astype(np.int64))
        gs = ws.stats()
        assert gs["trav_init"] == st["trav_init"]
        assert gs["relax_init"] == st["word_reach_deg"]
        assert gs["reached_init"] == st["word_reach_nodes"]
    assert gs["reached_init_t2"] > 0


def test_counts_by_snapshot_batch(im):
    insts = [(_graph(3000, 1500, 0.2, 4, ), 65, 2, 1), (_graph(900, 400, 0.5, 8), 200, 2, 2),
             (_graph(20000, 8000, 0.05, 6), 64, 2, 3)]
    dev = [(im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0"), R, k, s)
           for g, R, k, s in insts]
    for (g, R, k, s), (seeds, gains) in zip(insts, im.select_batch(dev)):
        s_ref, g_ref, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, R, k, s)
        assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
