"""Host logic of bench.py (CPU): the algorithmic bytes and counter figures of calls whose rounds run by
snapshot and of linear-threshold forests."""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def _stats():
    st = {"relax_fwd": 1000, "tasks_rev": 100}
    for p in ("init", "rev"):
        for t in range(3):
            st[f"relax_{p}_t{t}"] = 10000 * (t + 1)
            st[f"reached_{p}_t{t}"] = 100 * (t + 1)
            st[f"arcs_read_{p}_t{t}"] = 300 * (t + 1)
    return st


def test_bytes_by_snapshot_follow_live_heads():
    st = _stats()
    word, snap = bench.kernel_bytes(st, 50, 2), bench.kernel_bytes(st, 50, 2, covered=70)
    for ph in ("init_t0", "init_t1"):   # the same kernels either way
        assert word[ph] == snap[ph]
    assert word["rev_t1"] == 12 * 20000 + 16 * 200
    assert snap["rev_t1"] == 4 * 600 + 24 * 200
    assert snap["init_t2"] == 4 * 900 + 16 * 300
    assert snap["forward"] == (4 + 8 + 8 + 4 + 8) * 70
    # no figure of a search by snapshot depends on the degrees of what it reached
    for k in st:
        if k.startswith("relax_rev") or k in ("relax_fwd", "relax_init_t2"):
            st[k] *= 7
    assert bench.kernel_bytes(st, 50, 2, covered=70) == snap


def test_bytes_of_forests():
    b = bench.kernel_bytes_lt(1000, 64, 5000)
    assert set(bench.PROPAGATION) == set(b)
    assert b["init_t0"] == 36 * 64000 and b["forward"] == 36 * 5000 and b["rev_t1"] == 0


def test_rounds_are_told_by_the_packing_phase():
    assert bench.by_snapshot({"pack": (0.0, 0)}) and not bench.by_snapshot({"pack": (1.0, 50)})
    for ph in bench.SNAPSHOT_PHASES:
        assert bench.KERNEL_NAMES[ph] != bench.KERNEL_NAMES_SNAPSHOT[ph]


def test_counter_figures_of_kernels_by_snapshot(tmp_path, monkeypatch):
    src = tmp_path / "paper_1212_4779_amd" / "csrc"
    src.mkdir(parents=True)
    (src / "im_rev.h").write_text("x")
    (tmp_path / "profiles").mkdir()
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    rec = {"hbm_bytes_per_launch": 77, "sources": ["im_rev.h"], "source_digest": bench.source_digest(["im_rev.h"])}
    word = dict(rec, hbm_bytes_per_launch=99, kernel="void " + bench.kernel_signature("rev_t1", {}) + " x>")
    (tmp_path / "profiles" / "traffic.json").write_text(json.dumps(
        {"workloads": {"w": {"snapshot_kernels": {"rev_t1": rec}, "kernels": {"rev_t1": word}}}}))
    assert bench.load_traffic("rev_t1", "w", {}, snapshot=True) == 77
    assert bench.load_traffic("rev_t1", "w", {}) == 99
    assert bench.load_traffic("rev_t2", "w", {}, snapshot=True) is None
    (src / "im_rev.h").write_text("y")   # the kernel changed since
    assert bench.load_traffic("rev_t1", "w", {}, snapshot=True) is None
