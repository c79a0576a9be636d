"""Initial counts by snapshot with several tasks in progress per workgroup: graphs around the sizes
where the number of workgroups per CU, of wavefronts and of tasks in progress changes, with many
more large tasks than places; gains and counters against the oracle."""
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


@pytest.fixture(scope="module")
def core():
    """A near-critical graph, most of whose nodes reach hundreds of others, and its oracle gains."""
    g = gg.chung_lu_graph(4000, 40000, 2.5, 9, True, None)
    return g, *oracle.initial_gains(g.row_ptr, g.col, g.prob, 130, 5)


@pytest.mark.parametrize("n", [4000, 20767, 20769, 33505, 33537, 53279, 53281, 138337, 138369,
                               210241, 210273, 253952, 253985])
def test_tasks_in_progress(im, core, n):
    g, ref, st = core
    # nodes without arcs behind the graph change the sizes of the visited sets alone
    row_ptr = np.concatenate([g.row_ptr, np.full(n - g.n, g.m, np.uint64)])
    d = im.Graph.from_numpy(row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):
        got = im.initial_gains(d, 130, 5, ws=ws).cpu().numpy()
        assert np.array_equal(got[:g.n], ref.astype(np.int64)) and (got[g.n:] == 130).all()
        gs = ws.stats()
        assert gs["trav_init"] == st["trav_init"]
        assert gs["relax_init"] == st["word_reach_deg"]
        assert gs["reached_init"] == st["word_reach_nodes"] + 3 * (n - g.n)   # 130 snapshots: 3 words
    assert gs["reached_init_t2"] > 0


@pytest.mark.parametrize("leaves", [383, 384, 3071, 3072, 5000])
def test_table_limits(im, leaves):
    """Hubs of exactly the nodes that the tables of the first and second launch hold, and past them."""
    n = 260000
    row_ptr = np.concatenate([[0], np.full(n, leaves)]).astype(np.uint64)
    g = gg.Graph(n, row_ptr, np.arange(1, leaves + 1, dtype=np.uint32), np.ones(leaves, np.float32))
    ref, st = oracle.initial_gains(g.row_ptr, g.col, g.prob, 2, 5)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):   # the second call finds the marks as the first left them
        got = im.initial_gains(d, 2, 5, ws=ws).cpu().numpy()
        assert np.array_equal(got, ref.astype(np.int64))
        gs = ws.stats()
        assert gs["trav_init"] == st["trav_init"]
        assert gs["relax_init"] == st["word_reach_deg"]
        assert gs["reached_init"] == st["word_reach_nodes"]
    assert gs["reached_init_t2"] == leaves + 1


@pytest.mark.parametrize("leaves", [131040, 131104, 250000])
def test_marks_in_memory(im, leaves):
    """A hub whose 64 snapshots together touch fewer and more words of marks than are listed."""
    n = 260000
    row_ptr = np.concatenate([[0], np.full(n, leaves)]).astype(np.uint64)
    g = gg.Graph(n, row_ptr, np.arange(1, leaves + 1, dtype=np.uint32), np.full(leaves, 0.01, np.float32))
    ref, st = oracle.initial_gains(g.row_ptr, g.col, g.prob, 64, 5)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):   # the second call finds the marks as the first left them
        got = im.initial_gains(d, 64, 5, ws=ws).cpu().numpy()
        assert np.array_equal(got, ref.astype(np.int64))
        gs = ws.stats()
        assert gs["relax_init"] == st["word_reach_deg"]
        assert gs["reached_init"] == st["word_reach_nodes"]
