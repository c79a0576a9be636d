"""Linear-threshold rounds in which the wavefronts of a workgroup start far apart: thousands of
workgroups of 16 wavefronts compete for the device, and most seeds of the later rounds newly cover a
node or two, so that the wavefront which clears the first position of the interval is done at once.
Every wavefront has to have read that position before. Every round's gains against the oracle."""
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


@pytest.mark.parametrize("n,m,R,k", [(600, 3000, 4096, 40), (2000, 10000, 1024, 60)])
def test_every_wavefront_sees_the_uncovered_count(im, n, m, R, k):
    g = gg.chung_lu_graph(n, m, 2.5, 7, True, None)
    s_ref, g_ref, tr_ref = oracle.select_du_lt(g.row_ptr, g.col, g.prob, R, k, 3, trace=True)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    ws.set_live_edge(1)
    for _ in range(3):
        seeds, gains, tr = im.select(d, R, k, 3, ws=ws, trace=True)
        assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
        assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
