"""A workspace keeps buffers that a call can do without; on a device with little room left they are given
back when a later call needs the memory for what it cannot do without. A call that fits in no way is
an error, and leaves the workspace in order for the next one."""
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


def _lists(pair):
    return [x.cpu().tolist() for x in pair]


def _free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _dev(im, g):
    return im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")


R, K = 256, 4


def _calls(im, d, und):
    def threshold(ws):
        ws.set_live_edge(1)
        out = _lists(im.select(d, 128, K, 3, ws=ws)[:2])
        ws.set_live_edge(0)
        return out
    return [lambda ws: _lists(im.select(d, R, K, 3, ws=ws)[:2]),
            lambda ws: _lists(im.select_lazy(d, R, K, 3, ws=ws)),
            threshold,
            lambda ws: _lists(im.select_undirected(und, 64, K, 3, ws=ws)[:2]),
            lambda ws: _lists(im.select_batch([(d, R, K, 3), (d, 64, K, 4)], ws=ws)[0])]


def test_calls_in_any_order_with_little_room(im):
    import torch
    d = _dev(im, gg.chung_lu_graph(1_000_000, 2_000_000, 2.3, 31, True, 0.05))
    und = _dev(im, gg.chung_lu_graph(1_000_000, 2_000_000, 2.3, 33, False, 0.05))
    calls = _calls(im, d, und)
    refs = []
    for on in (0, 1):   # (also: every kernel has run once before memory gets short)
        refs = []
        for c in calls:
            ws = im.Workspace()
            ws.set_max_slots(8)
            ws.set_sparse_lists(on)
            refs.append(c(ws))
            ws.close()
    assert refs[0] == refs[1] == refs[4]
    small = gg.chung_lu_graph(700, 4000, 2.4, 35, True, None)
    s, gn, _, _ = oracle.select_du(small.row_ptr, small.col, small.prob, 100, 5, 9)
    huge = torch.zeros(40_000_001, dtype=torch.int64, device="cuda:0")
    none = torch.empty(0, device="cuda:0")
    huge = im.Graph(huge, none.to(torch.int32), none)
    small = _dev(im, small)
    hold = torch.empty(_free() - int(4.6 * 2**30), dtype=torch.uint8, device="cuda:0")
    try:
        ws = im.Workspace()
        ws.set_max_slots(8)
        for i in (0, 1, 3, 0, 2, 4, 1):
            assert calls[i](ws) == refs[i], i
        # 40 million nodes do not fit: an error, and then the workspace serves calls as before
        for call in (lambda: im.select(huge, 64, 2, 1, ws=ws),
                     lambda: im.select_undirected(huge, 64, 2, 1, ws=ws)):
            with pytest.raises(im.ImError, match="hipMalloc"):
                call()
            assert _lists(im.select(small, 100, 5, 9, ws=ws)[:2]) == [s.tolist(), gn.tolist()]
            assert _lists(im.select_lazy(small, 100, 5, 9, ws=ws)) == [s.tolist(), gn.tolist()]
        assert calls[3](ws) == refs[3]
        ws.close()
    finally:
        del hold
        torch.cuda.empty_cache()
