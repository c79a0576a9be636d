"""Linear threshold at almost 2^32 (node, snapshot) pairs, where the launches that give every pair a
lane would hold 2^32 lanes once the snapshots are rounded up: such a call runs the general engines.
A path of 1,000 nodes whose arcs are always kept, and isolated nodes."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def im():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4779_amd as im
    return im


@pytest.mark.parametrize("n,R", [(1048576, 4088), (1048832, 4095)])
def test_most_pairs(im, n, R):
    import torch
    row = torch.full((n + 1,), 999, dtype=torch.int64, device="cuda:0")
    row[:1000] = torch.arange(1000)
    col = torch.arange(1, 1000, dtype=torch.int32, device="cuda:0")
    d = im.Graph(row, col, torch.ones(999, dtype=torch.float32, device="cuda:0"))
    ws = im.Workspace()
    ws.set_live_edge(1)
    seeds, gains, _ = im.select(d, R, 3, 5, ws=ws)
    assert seeds.cpu().tolist() == [0, 1000, 1001] and gains.cpu().tolist() == [1000 * R, R, R]
    ws.close()
