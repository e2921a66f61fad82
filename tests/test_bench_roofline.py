"""The bench's roofline: which kernel it names and what it counts, from the launches
of the timer classes."""
import importlib.util
import os

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def bench():
    spec = importlib.util.spec_from_file_location("bench", os.path.join(ROOT, "bench.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def test_node_update_reads_the_cells_products():
    # 10 applies in 10 steps, 9 of them recurrence steps; 2 ms an update
    t = {"cell": (10, 8.0), "pre": (10, 20.0), "recur": (9, 40.0)}
    r = bench().roofline("fp64", 160, 343, 4096, 912673, t)
    want = 8 * 160 * (343 * 4096 + 912673 * (1 + 2.7))
    assert r["bound"] == "hbm" and r["kernel"] == "k_node_update"
    assert abs(r["bytes_per_launch"] - want) < 1e-6 * want
    assert abs(r["achieved"] - want / 2e-3 / 1e12) < 1e-9 * r["achieved"]


def test_dense_cells_are_a_colour_pass():
    # BF16: the node update reads no products, eight launches of cells an apply
    t = {"cell": (80, 40.0), "pre": (10, 20.0), "recur": (9, 60.0)}
    r = bench().roofline("bf16", 160, 343, 4096, 912673, t)
    want = 2 * 343 ** 2 * 4096 * 160 / 8
    assert r["bound"] == "mfma" and "colour" in r["kernel"] and "bytes_per_launch" not in r
    assert abs(r["flops_per_launch"] - want) < 1e-6 * want
    assert abs(r["frac"] - want / 0.5e-3 / 2.5e15) < 1e-9


def test_traffic_is_of_this_source_and_precision(tmp_path, monkeypatch):
    import hashlib
    import json
    m = bench()
    monkeypatch.setattr(m, "ROOT", str(tmp_path))
    src = tmp_path / "paper_2607_06848_amd" / "csrc" / "apply.hip"
    src.parent.mkdir(parents=True)
    src.write_text("a")
    assert m.measured_traffic("k_node_update", "c64", "fp64") is None
    rec = {"apply_hip_sha256": hashlib.sha256(b"a").hexdigest(), "prec": "fp64",
           "kernels": {"k_node_update": {"read_bytes": 5.0, "write_bytes": 2.0}}}
    (tmp_path / "profiles").mkdir()
    (tmp_path / "profiles" / "node_update_c64_traffic.json").write_text(json.dumps(rec))
    assert m.measured_traffic("k_node_update", "c64", "fp64") == 7.0
    assert m.measured_traffic("k_node_update", "c64", "fp32") is None
    src.write_text("b")
    assert m.measured_traffic("k_node_update", "c64", "fp64") is None
