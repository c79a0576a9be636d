"""One workspace through calls of both snapshot models: what a linear-threshold call leaves on it
(buffers sized for that graph, the rounds on forests) does not reach the batched or single calls that
follow, and the other way round. Seeds and gains against the oracle."""
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


def _dev(im, g):
    return im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")


def _lists(pair):
    return [x.cpu().tolist() for x in pair]


def _instances(im):
    """Larger together, and each, than the linear-threshold graph before them."""
    insts, refs = [], []
    for i, (n, p) in enumerate(((900, None), (2500, 0.05), (1300, None))):
        g = gg.chung_lu_graph(n, n * 6, 2.5, 300 + i, True, p)
        R, k = (100, 64, 130)[i], 4 + i
        insts.append((_dev(im, g), R, k, 11 + i))
        s, gn, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, R, k, 11 + i)
        refs.append([s.tolist(), gn.tolist()])
    return insts, refs


def _threshold_call(im, ws, valid):
    g = gg.chung_lu_graph(200, 1200, 2.5, 7, True, None)
    d = _dev(im, g)
    ws.set_live_edge(1)
    if valid:
        s, gn, _ = oracle.select_du_lt(g.row_ptr, g.col, g.prob, 64, 6, 3, trace=True)
        assert _lists(im.select(d, 64, 6, 3, ws=ws)[:2]) == [s.tolist(), gn.tolist()]
    else:
        d.prob.fill_(2.0)   # no probability: refused by the validation kernel
        with pytest.raises(im.ImError):
            im.select(d, 64, 6, 3, ws=ws)
    ws.set_live_edge(0)


@pytest.mark.parametrize("valid", [True, False])
@pytest.mark.parametrize("tuned", [False, True])
def test_batch_after_a_linear_threshold_call(im, valid, tuned):
    insts, refs = _instances(im)
    ws = im.Workspace()
    _threshold_call(im, ws, valid)
    if tuned:
        im.autotune_batch(insts, ws=ws)
    assert [_lists(x) for x in im.select_batch(insts, ws=ws)] == refs
    # and back: each model again on the workspace that the other one used
    _threshold_call(im, ws, True)
    (d, R, k, seed), ref = insts[1], refs[1]
    assert _lists(im.select(d, R, k, seed, ws=ws)[:2]) == ref
    assert _lists(im.select_lazy(d, R, k, seed, ws=ws)) == ref
    assert [_lists(x) for x in im.select_batch(insts, ws=ws)] == refs
