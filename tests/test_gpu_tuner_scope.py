"""What the tuner's choice applies to: the snapshot model it was timed on, and the engines of this
library (cache lines of earlier formats are passed over)."""
import json
import os
import subprocess
import sys

import pytest

import oracle
from paper_1212_4779_amd import graphgen as gg

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def im():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1212_4779_amd as im
    return im


def _dev(im, g):
    return im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device="cuda:0")


def test_choice_per_snapshot_model(im):
    g = gg.chung_lu_graph(900, 5000, 2.5, 81, True, None)
    d = _dev(im, g)
    ws = im.Workspace()
    ws.set_live_edge(1)
    t = im.autotune(d, 70, 3, ws=ws)
    assert t["tried"] == 1 and t["affected_gain"] == 0   # forests read no schedule
    assert im.autotune(d, 70, 3, ws=ws)["tried"] == 0
    s, gn, _ = oracle.select_du_lt(g.row_ptr, g.col, g.prob, 70, 5, 3, trace=True)
    seeds, gains, _ = im.select(d, 70, 5, 3, ws=ws)
    assert [seeds.cpu().tolist(), gains.cpu().tolist()] == [s.tolist(), gn.tolist()]
    ws.set_live_edge(0)
    t = im.autotune(d, 70, 3, ws=ws)
    assert t["tried"] >= 2
    s, gn, _, _ = oracle.select_du(g.row_ptr, g.col, g.prob, 70, 5, 3)
    seeds, gains, _ = im.select(d, 70, 5, 3, ws=ws)
    assert [seeds.cpu().tolist(), gains.cpu().tolist()] == [s.tolist(), gn.tolist()]


def test_knobs_that_nothing_reads_are_not_timed(im):
    g = gg.chung_lu_graph(1100, 6000, 2.5, 82, True, 0.05)
    d = _dev(im, g)
    t = im.autotune(d, 64, 3, ws=im.Workspace())
    if t["affected_gain"] == 0:   # rounds by snapshot: seven schedules, four update strategies
        assert t["tried"] == 7 + 4 and t["coop_forward"] == 1
    ws = im.Workspace()
    ws.set_sparse_lists(0)
    h = gg.chung_lu_graph(1000, 6000, 2.5, 83, True, 0.05)
    assert im.autotune(_dev(im, h), 64, 3, ws=ws)["tried"] >= 10 + 4 + 4   # rounds by word: all


def test_lines_of_earlier_engines_are_passed_over(im, tmp_path):
    cache = tmp_path / "tune.txt"
    code = ("import json, sys; sys.path.insert(0, %r)\n"
            "import paper_1212_4779_amd as im\n"
            "from paper_1212_4779_amd import graphgen as gg\n"
            "g = gg.workload_graph('tiny_uic')\n"
            "d = im.Graph.from_numpy(g.row_ptr, g.col, g.prob, device='cuda:0')\n"
            "print(json.dumps(im.autotune(d, 64, 1)))\n" % ROOT)

    def run():
        r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, IM_TUNE_CACHE=str(cache)),
                           capture_output=True, text=True, timeout=240)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout.strip().splitlines()[-1])

    assert run()["tried"] > 0
    line = cache.read_text().splitlines()[0].split()
    assert len(line) == 17 and line[-2:] == ["0", "2"]
    old = line[:10] + [str(1 << 62)] + line[11:15]           # without model and engines
    other = line[:10] + [str(1 << 62)] + line[11:15] + ["0", "1"]
    cache.write_text(" ".join(old) + "\n" + " ".join(other) + "\n")
    t = run()
    assert t["tried"] > 0   # tuned again, and appended
    assert len(cache.read_text().splitlines()) == 3
    assert run()["tried"] == 0
