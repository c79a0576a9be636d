"""The linear-threshold dynamic update on forests: cycles, self-loops, weights of zero and past one,
and in-rows around the sizes where the sort changes (64 in-arcs, the workgroup's tile), against the
oracle and, for the counters, against the definitions on the trace."""
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


def _ring(n):
    """One cycle through every node (all weights one), with a tail."""
    src = list(range(n)) + [3]
    dst = [(i + 1) % n for i in range(n)] + [n]
    return _graph(n + 1, src, dst, [1.0] * (n + 1))


def _rows(d, rng):
    """Three heads of d - 1, d and d + 1 in-arcs, duplicates among them, with zero weights and
    sums past one; the heads feed each other and themselves."""
    n = 3 * d
    src, dst, w = [], [], []
    for h, deg in enumerate((d - 1, d, d + 1)):
        tails = rng.integers(0, n, deg)
        tails[0] = h                       # a self-loop
        tails[-1] = (h + 1) % 3            # heads in a cycle
        src += tails.tolist()
        dst += [h] * deg
        x = rng.random(deg) * (2.2 / deg)
        x[rng.random(deg) < 0.2] = 0.0
        w += x.tolist()
    # and a random sparse rest
    m = 2 * n
    src += rng.integers(0, n, m).tolist()
    dst += rng.integers(3, n, m).tolist()
    w += (rng.random(m) * 0.5).tolist()
    return _graph(n, src, dst, np.minimum(w, 1.0))


def _cases():
    rng = np.random.default_rng(5)
    out = [("ring", _ring(700), 3, 4), ("no_arcs", _graph(5, [], [], []), 65, 3),
           ("loops", _graph(4, [0, 1, 2, 3], [0, 1, 2, 3], [1.0, 0.5, 0.0, 1.0]), 64, 4)]
    for d in (64, 65, 512, 513, 1300):
        out.append((f"rows_{d}", _rows(d, rng), 70, 6))
    n = 1500   # a random mapping: many cycles and deep trees
    out.append(("mapping", _graph(n, rng.integers(0, n, n), rng.permutation(n), [1.0] * n), 5, 12))
    return out


@pytest.mark.parametrize("case", _cases(), ids=lambda c: c[0])
def test_forest_rounds(im, case):
    _, g, R, k = case
    seed = 17
    s_ref, g_ref, tr_ref = oracle.select_du_lt(g.row_ptr, g.col, g.prob, R, k, seed, trace=True)
    d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")
    ws = im.Workspace()
    ws.set_live_edge(1)
    for _ in range(2):   # the second call finds the buffers as the first left them
        seeds, gains, tr = im.select(d, R, k, seed, ws=ws, trace=True)
        assert seeds.cpu().tolist() == s_ref.tolist() and gains.cpu().tolist() == g_ref.tolist()
        assert np.array_equal(tr.cpu().numpy().astype(np.uint32), tr_ref)
    st = ws.stats()
    assert st["decrements"] == int(tr_ref[0].astype(np.int64).sum() - tr_ref[k].astype(np.int64).sum())
    # the traversal counters against the per-snapshot definition
    live = oracle.live_bits_lt(g.row_ptr, g.col, g.prob, R, seed)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr.astype(np.int64)))
    out_deg, in_deg = g.out_degree(), g.in_degree()
    want = dict(trav_init=0, trav_fwd=0, trav_rev=0)
    for r in range(min(R, 6)) if R <= 6 else ():
        on = ((live[:, r // 64] >> np.uint64(r % 64)) & np.uint64(1)).astype(bool)
        children = [[] for _ in range(g.n)]
        for a, b in zip(src[on], g.col[on]):
            children[a].append(int(b))
        reach = []
        for u in range(g.n):
            seen, todo = {u}, [u]
            while todo:
                for y in children[todo.pop()]:
                    if y not in seen:
                        seen.add(y)
                        todo.append(y)
            reach.append(seen)
        want["trav_init"] += sum(int(out_deg[x]) for s in reach for x in s)
        covered = set()
        for v in s_ref.tolist():
            new = reach[v] - covered
            covered |= new
            want["trav_fwd"] += sum(int(out_deg[x]) for x in new)
            want["trav_rev"] += sum(int(in_deg[y]) * len(reach[y] & new) for y in range(g.n))
    if R <= 6:
        assert {key: st[key] for key in want} == want
