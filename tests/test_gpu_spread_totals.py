"""Marginals whose share of one workgroup passes 2^32. Graphs this large leave the spread evaluator a
few workgroups (the queues of n words each stay within a budget), which take the snapshots in turn.
A star whose arcs are all live: the hub covers every node in every snapshot, the second seed nothing."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def im():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4779_amd as im
    return im


def test_marginals_past_32_bits(im):
    import torch
    n, R = 2048 * 244_141, 17   # two workgroups: nine snapshots, 4.5 * 10^9 nodes, and eight
    row = torch.full((n + 1,), n - 1, dtype=torch.int64, device="cuda:0")
    row[0] = 0
    # consecutive arcs lead to consecutive words of the bitmap (to one word they would queue there)
    col = torch.arange(n, dtype=torch.int32, device="cuda:0")
    col = col.view(-1, 32, 64).transpose(1, 2).reshape(-1)[1:].contiguous()
    d = im.Graph(row, col, torch.ones(n - 1, dtype=torch.float32, device="cuda:0"))
    seeds = torch.tensor([0, 5], device="cuda:0")
    ws = im.Workspace()
    marg, per = im.spread(d, R, 3, seeds, ws=ws, per_snapshot=True)
    assert per.cpu().tolist() == [n] * R
    assert marg.cpu().tolist() == [n * R, 0]
    ws.close()
    del row, col, d, marg, per
    torch.cuda.empty_cache()
