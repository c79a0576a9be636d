"""Spread evaluation on small graphs of many arcs, where the lanes per snapshot go by arcs and
snapshots: both sides of the lines, with the marginals and for the whole set at once, against the oracle."""
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


@pytest.mark.parametrize("n,m,p,R,nS", [
    (3000, 131071, 0.05, 9, 20), (3000, 131072, 0.05, 9, 20), (3000, 131072, 0.05, 1, 300),
    (3000, 140000, 0.002, 1023, 5), (3000, 140000, 0.002, 1024, 5), (3000, 140000, 0.002, 8191, 3),
    (3000, 140000, 0.002, 8192, 3), (16384, 200000, 0.03, 65, 12), (16385, 200000, 0.03, 65, 12)])
def test_spread_by_arcs(im, n, m, p, R, nS):
    g = gg.chung_lu_graph(n, m, 2.5, 51, True, p)
    S = np.random.default_rng(n + R).integers(0, n, nS).astype(np.uint32)
    marg_ref, per_ref = oracle.spread_prefix(g.row_ptr, g.col, g.prob, R, 7, S)
    import torch
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    seeds = torch.from_numpy(S.astype(np.int64)).to("cuda:0")
    ws = im.Workspace()
    marg, per = im.spread(d, R, 7, seeds, ws=ws, per_snapshot=True)
    assert marg.cpu().tolist() == marg_ref.tolist() and per.cpu().tolist() == per_ref.tolist()
    _, per = im.spread(d, R, 7, seeds, ws=ws, marginals=False, per_snapshot=True)
    assert per.cpu().tolist() == per_ref.tolist()
