"""Lazy evaluations and commits by snapshot: visit bits in LDS or in memory (2^18 nodes), queues past
their LDS parts (2,048 entries in an evaluation, 4,096 in a commit), a seed evaluated in an earlier
batch of its round (batch 1), and a batch whose queues exceed the budget (by word), against the oracle."""
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


def _stars(n, leaves, p, seed):
    """Overlapping stars of the given sizes (shared leaves), a path behind every leaf."""
    rng = np.random.default_rng(seed)
    hubs = len(leaves)
    pool = rng.permutation(np.arange(hubs, n))[:2 * max(leaves)]
    src, dst = [], []
    for h, size in enumerate(leaves):
        src += [h] * size
        dst += rng.choice(pool, size, replace=False).tolist()
    src += pool[:-1].tolist()
    dst += pool[1:].tolist()
    src, dst = np.array(src, np.int64), np.array(dst, np.int64)
    row_ptr, col = gg.to_csr(n, src, dst)
    tails = np.repeat(np.arange(n), np.diff(row_ptr.astype(np.int64)))
    return gg.Graph(n, row_ptr, col, np.where(tails < hubs, p, 0.2).astype(np.float32))


@pytest.mark.parametrize("n,leaves,p,R,k,batch", [
    (9000, (2040, 2060, 1500, 900), 0.999, 66, 5, 3), (20000, (5200, 4100, 4090, 60), 0.99, 3, 5, 1),
    (262144, (2500, 1200, 5000), 0.9, 5, 4, 2), (262145, (2500, 1200, 5000), 0.9, 5, 4, 2),
    (262145, (2500, 1200, 5000), 0.9, 65, 4, 1), (262145, (800, 700, 600), 0.5, 64, 4, 300),
])
def test_lazy_by_snapshot(im, n, leaves, p, R, k, batch):
    g = _stars(n, leaves, p, 3)
    s_ref, g_ref, st = oracle.select_celf(g.row_ptr, g.col, g.prob, R, k, 7)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    for _ in range(2):   # the second call finds the visit bits as the first left them
        seeds, gains = im.select_lazy(d, R, k, 7, batch=batch, ws=ws)
        assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
    if batch == 1:
        assert ws.stats()["celf_evals"] == st["celf_evals"]
