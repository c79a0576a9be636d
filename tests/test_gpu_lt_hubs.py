"""Linear-threshold forests in which the leaves of a wavefront share their parents: stars, hubs dealt in
turn (groups of every size down to lanes that are alone), a hub whose leaves fill
parts of wavefronts, and hubs below other hubs; every round's gains against the oracle."""
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


def _graph(n, src, dst, w):
    src, dst, w = np.asarray(src, np.int64), np.asarray(dst, np.int64), np.asarray(w, np.float32)
    order = np.argsort(src, kind="stable")
    row_ptr = np.zeros(n + 1, np.uint64)
    row_ptr[1:] = np.cumsum(np.bincount(src, minlength=n))
    return gg.Graph(n, row_ptr, dst[order].astype(np.uint32), w[order])


def _dealt(hubs, leaves, w):
    """`leaves` leaves dealt to the hubs in turn; the hubs themselves hang from hub 0."""
    n = hubs + leaves
    leaf = np.arange(hubs, n)
    src = np.concatenate([leaf % hubs, np.zeros(hubs - 1, np.int64)])
    dst = np.concatenate([leaf, np.arange(1, hubs)])
    return _graph(n, src, dst, np.full(len(src), w))


def _blocks(sizes, w):
    """Hubs of the given numbers of leaves, one after another, each hub the child of the one before it."""
    src, dst, at, last = [], [], 0, -1
    for s in sizes:
        if last >= 0:
            src.append(last), dst.append(at)
        last = at
        src += [at] * s
        dst += list(range(at + 1, at + 1 + s))
        at += 1 + s
    return _graph(at, src, dst, np.full(len(src), w))


@pytest.mark.parametrize("g,R", [
    (_dealt(1, 1000, 0.5), 70), (_dealt(1, 63, 1.0), 9), (_dealt(15, 2000, 0.7), 65), (_dealt(16, 2000, 1.0), 64),
    (_dealt(17, 2000, 1.0), 64), (_dealt(22, 2000, 0.6), 33), (_dealt(300, 3000, 0.9), 20),
    (_blocks([3, 4, 5, 63, 64, 65, 127, 1, 200], 0.9), 130), (_blocks([4] * 60, 1.0), 8)],
    ids=lambda x: str(x) if isinstance(x, int) else f"{x.n}_{x.m}")
def test_leaves_of_one_parent(im, g, R):
    k = 8
    s_ref, g_ref, tr_ref = oracle.select_du_lt(g.row_ptr, g.col, g.prob, R, k, 3, trace=True)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    ws.set_live_edge(1)
    seeds, gains, tr = im.select(d, R, k, 3, ws=ws, trace=True)
    assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
    assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
