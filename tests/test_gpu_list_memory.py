"""The per-snapshot live lists take memory by the snapshots asked for, and a call whose lists (or the
other buffers that it can do without) do not fit beside another holder of the device's memory runs
without them: same seeds and gains."""
import numpy as np
import pytest

from paper_1212_4779_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def im():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4779_amd as im
    return im


def _free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _lists(pair):
    return [x.cpu().tolist() for x in pair]


def test_memory_of_one_snapshot(im):
    import torch
    n, m = 16_000_000, 1000
    row = torch.full((n + 1,), m, dtype=torch.int64, device="cuda:0")
    row[:m] = torch.arange(m)
    col = torch.arange(1, m + 1, dtype=torch.int32, device="cuda:0")
    d = im.Graph(row, col, torch.ones(m, dtype=torch.float32, device="cuda:0"))
    used = {}
    for on in (0, 1):
        ws = im.Workspace()
        ws.set_sparse_lists(on)
        before = _free()
        seeds, gains, _ = im.select(d, 1, 2, 5, ws=ws)
        used[on] = before - _free()
        assert _lists((seeds, gains)) == [[0, m + 1], [m + 1, 1]]
        ws.close()
    # lists of both directions, newly covered nodes and stamps of the rounds by snapshot: 16 bytes
    # per node (and a closing offset per 256), and at most 4 GB for the initial counts
    assert used[1] - used[0] <= 17 * n + (4 << 30) + (64 << 20)


@pytest.fixture(scope="module")
def big(im):
    g = gg.chung_lu_graph(1_000_000, 2_000_000, 2.3, 31, True, 0.05)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ref = []
    for on in (0, 1):   # (also: every kernel has run once before memory gets short)
        ws = im.Workspace()
        ws.set_sparse_lists(on)
        ws.set_max_slots(8)
        ref.append([_lists(im.select(d, 256, 6, 3, ws=ws)[:2]), _lists(im.select_lazy(d, 256, 6, 3, ws=ws))])
        ws.close()
    assert ref[0] == ref[1] and ref[0][0] == ref[0][1]
    return d, ref[0][0]


# about 1.1 GB that the call needs, 1.5 for the lists of each direction, 1.1 for the rounds by
# snapshot and 0.5 for the initial counts: none, one or both lists, all of it
@pytest.mark.parametrize("left", [2.0, 3.2, 4.6, 9.0])
def test_call_beside_another_holder(im, big, left):
    import torch
    d, ref = big
    hold = torch.empty(_free() - int(left * 2**30), dtype=torch.uint8, device="cuda:0")
    try:
        for call in (lambda ws: im.select(d, 256, 6, 3, ws=ws)[:2],
                     lambda ws: im.select_lazy(d, 256, 6, 3, ws=ws)):
            ws = im.Workspace()
            ws.set_max_slots(8)
            out = _lists(call(ws))
            ws.close()
            assert out == ref
    finally:
        del hold
        torch.cuda.empty_cache()
    assert np.all(np.diff(ref[1]) <= 0)
