"""Batches around the most workgroups that one launch of the forward step by snapshot can hold
(instances times snapshots, 512 lanes each, below 2^32 lanes): one instance fewer runs by snapshot,
at the bound and past it the rounds run by word. Every instance against the oracle."""
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


@pytest.mark.parametrize("count", [8191, 8192, 8200])
def test_many_small_instances(im, count):
    R, k = 1024, 3
    insts, refs = [], []
    for i in range(4):
        g = gg.chung_lu_graph(16 + i, 40, 2.5, 400 + i, True, (0.1, 0.4, None, 1.0)[i])
        insts.append((im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0"), R, k, 5 + i))
        s, gn, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, R, k, 5 + i)
        refs.append((s.tolist(), gn.tolist()))
    ws = im.Workspace()
    out = im.select_batch([insts[i % 4] for i in range(count)], ws=ws)
    import torch
    seeds = torch.stack([s for s, _ in out]).cpu().numpy()
    gains = torch.stack([g for _, g in out]).cpu().numpy()
    for i in range(4):
        assert np.array_equal(seeds[i::4], np.tile(refs[i][0], (len(seeds[i::4]), 1)))
        assert np.array_equal(gains[i::4], np.tile(refs[i][1], (len(gains[i::4]), 1)))
    ws.close()
