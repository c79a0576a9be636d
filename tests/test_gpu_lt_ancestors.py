"""Linear-threshold rounds whose seed has many ancestors (64 are taken at a time), with and without
a cycle above them, and row counts that do not fill the last group of snapshots; seeds, gains and
every round's gains against the oracle."""
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


def _graph(path, ring):
    """`ring` nodes in a cycle, a path of `path` nodes from it (arcs of weight 0.995) and 400
    leaves at its end, which is the first seed."""
    src, dst, w = [], [], []
    for i in range(ring):
        src.append(i), dst.append((i + 1) % ring), w.append(1.0)
    end = ring + path - 1
    for i in range(max(ring - 1, 0), end):
        src.append(i), dst.append(i + 1), w.append(0.995)
    for i in range(400):
        src.append(end), dst.append(end + 1 + i), w.append(1.0)
    n = end + 401
    src, dst, w = np.array(src), np.array(dst), np.array(w, np.float32)
    order = np.argsort(src, kind="stable")
    row_ptr = np.zeros(n + 1, np.uint64)
    row_ptr[1:] = np.cumsum(np.bincount(src, minlength=n))
    return gg.Graph(n, row_ptr, dst[order].astype(np.uint32), w[order])


@pytest.mark.parametrize("path,ring,R", [(1, 0, 3), (64, 0, 9), (65, 0, 65), (66, 0, 70), (129, 0, 128),
                                         (2, 63, 9), (2, 64, 9), (2, 65, 65), (400, 1, 130)])
def test_ancestors(im, path, ring, R):
    g = _graph(path, ring)
    s_ref, g_ref, tr_ref = oracle.select_du_lt(g.row_ptr, g.col, g.prob, R, 5, 3, trace=True)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    ws.set_live_edge(1)
    seeds, gains, tr = im.select(d, R, 5, 3, ws=ws, trace=True)
    assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
    assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
