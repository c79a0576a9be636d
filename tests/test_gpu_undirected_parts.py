"""The component method's initial gains with the snapshots split over workgroups: node counts around
the sizes where the split begins and ends, snapshot counts around its steps, against the oracle."""
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


@pytest.mark.parametrize("n,R", [(200, 1), (300, 7), (300, 8), (300, 9), (3560, 230), (30000, 65),
                                 (131073, 17), (261888, 9), (261889, 9)])
def test_split_gains(im, n, R):
    g = gg.chung_lu_graph(max(min(n, 3000), 2), max(min(3 * n, 9000), 2), 2.5, 4, False, 0.1)
    row_ptr = np.concatenate([g.row_ptr, np.full(n - g.n, g.m, np.uint64)])
    g = gg.Graph(n, row_ptr, g.col, g.prob)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    k = min(n, 4)
    s_ref, g_ref, tr_ref = oracle.select_components(g.row_ptr, g.col, g.prob, R, k, 6, trace=True)
    ws = im.Workspace()
    for _ in range(2):
        seeds, gains, tr = im.select_undirected(d, R, k, 6, ws=ws, trace=True)
        assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
        assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
