"""The spread evaluator at the sizes where it changes: lanes per snapshot (16,384 nodes, 1,024
snapshots), visit bits in LDS or in global memory (2^18 nodes), marginals added up per workgroup
(256 seeds), against the oracle."""
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
    (16384, 40000, 0.2, 70, 257), (16385, 40000, 0.2, 1023, 12), (16385, 40000, None, 1024, 256),
    (262144, 300000, 0.3, 3, 40), (262145, 300000, 0.3, 3, 40), (262145, 300000, 0.3, 1024, 2),
    (5000, 20000, 1.0, 65, 3), (5000, 20000, 0.0, 65, 3),
])
def test_spread_sizes(im, n, m, p, R, nS):
    g = gg.chung_lu_graph(n, m, 2.4, 3, True, p)
    rng = np.random.default_rng(n + R)
    S = [int(np.argmax(g.out_degree()))] + [int(x) for x in rng.integers(0, n, nS - 1)]
    marg_ref, per_ref = oracle.spread_prefix(g.row_ptr, g.col, g.prob, R, 9, S)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):   # the second call finds the visit bits as the first left them
        marg, per = im.spread(d, R, 9, S, ws=ws, per_snapshot=True)
        assert marg.cpu().tolist() == marg_ref.tolist() and per.cpu().tolist() == per_ref.tolist()
    _, per = im.spread(d, R, 9, S, ws=ws, marginals=False, per_snapshot=True)
    assert per.cpu().tolist() == per_ref.tolist()
