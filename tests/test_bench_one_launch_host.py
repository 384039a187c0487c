"""The bench's roofline of solves in one launch: which solves those are, the
bytes their iterations stream, and counter traffic tied to that kernel's own
sources (bench.py; no GPU)."""
import json
import os

import bench


def test_bytes_streamed():
    # a periodic Kuhn cube: 14 neighbours a node, 6 tetrahedra a node, V + T = 7 V edges
    v = 46 ** 3
    assert bench.rows_iteration_bytes(v, 6 * v, 4, 1, True) == 14 * v * 6 + 4 * v
    assert bench.rows_iteration_bytes(v, 6 * v, 8, 6, False) == 14 * v * 50


def test_limits_follow_rows_per_workgroup():
    for n, gs32, gs64, el in ((729, 1, 1, 1), (262144, 1, 1, 1), (262145, 1, 1, 0), (524288, 1, 1, 0),
                              (524289, 1, 0, 0), (1048576, 1, 0, 0), (1048577, 0, 0, 0)):
        got = (bench.one_launch(n, True, False), bench.one_launch(n, False, False), bench.one_launch(n, True, True))
        assert got == (bool(gs32), bool(gs64), bool(el)), n


def test_traffic_of_its_own_sources(tmp_path, monkeypatch):
    path, sources = bench.TRAFFIC["gs_one_launch"]
    assert any(f.endswith("resident_kernel.h") for f in sources)
    with open(os.path.join(bench.ROOT, path)) as f:
        t = json.load(f)
    t["kernel_hash"] = bench.kernel_hash("gs_one_launch")
    tmp = tmp_path / "t.json"
    tmp.write_text(json.dumps(t))
    monkeypatch.setitem(bench.TRAFFIC, "gs_one_launch", (str(tmp), sources))
    assert bench.traffic_from_profile("gs_one_launch", "mixed+precond") == t["mixed+precond"]["bytes_per_launch"]
    t["kernel_hash"] = "0" * 16
    tmp.write_text(json.dumps(t))
    assert bench.traffic_from_profile("gs_one_launch", "mixed+precond") is None
