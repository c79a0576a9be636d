"""Buffers that a call can do without leave the device a gigabyte: kernels with private memory get it
when they are launched. Beside another holder of the memory, every kind of call ends with that much
left, and with the results that it has when alone."""
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


def _lists(pair):
    return [x.cpu().tolist() for x in pair]


def _free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def _select(im, d, ws, R):
    return _lists(im.select(d, R, 4, 3, ws=ws)[:2])


def _threshold(im, d, ws, R):
    ws.set_live_edge(1)
    return _select(im, d, ws, R)


def _lazy(im, d, ws, R):
    return _lists(im.select_lazy(d, R, 4, 3, ws=ws))


def _batch(im, d, ws, R):
    return _lists(im.select_batch([(d, R, 4, 3), (d, 64, 4, 4)], ws=ws)[0])


def test_room_is_left(im):
    import torch
    g = gg.chung_lu_graph(1_000_000, 2_000_000, 2.3, 31, True, 0.05)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")

    def call(f, R, on=1):
        ws = im.Workspace()
        ws.set_max_slots(8)
        ws.set_sparse_lists(on)
        out = f(im, d, ws, R)
        left = _free()
        ws.close()
        return out, left

    kinds = (_select, _threshold, _lazy, _batch)
    # about 1.1 GB is needed (two for the batch), the rest could take 4 (select) to 12 GB
    refs = {(f, R): call(f, R)[0] for f in kinds for R in (128, 256)}
    for f in kinds:   # (the other engines' kernels have run once, too)
        assert call(f, 256, 0)[0] == refs[f, 256]
    hold = torch.empty(_free() - (5 << 30), dtype=torch.uint8, device="cuda:0")
    try:
        for (f, R), ref in refs.items():
            out, left = call(f, R)
            assert out == ref, (f.__name__, R)
            assert left >= 1 << 30, (f.__name__, R, left)
    finally:
        del hold
        torch.cuda.empty_cache()
