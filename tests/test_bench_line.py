"""bench.py's result line: one line of JSON short enough to be kept whole, with
everything that the benchmark's contract names; the tables that do not fit go
to the details file alone."""
from __future__ import annotations

import json

import bench

CONTRACT = {"metric": "m", "value": 3245.12, "unit": "TOPS", "n_gpus": 1, "steps": 20, "warmup": 5,
            "ms_per_step": 15.586, "step_ms": [15.57] * 20, "higher_is_better": True, "scaling": "weak",
            "vs_baseline": None, "dtype": "i8", "data": "synthetic", "config": {"n": 8192, "iters": [8] * 9},
            "roofline": {"bound": "mfma", "achieved": 3281.5}}


def _rows(count, keys):
    return [{f"some_quantity_{k}": 1234.5678 + i for k in range(keys)} for i in range(count)]


def _full(scale):
    return {**CONTRACT, "per_graph": _rows(9 * scale, 7),
            "extras": {"autotune": _rows(10 * scale, 5), "tc_plain_fp32": _rows(9 * scale, 8),
                       "tc_square_variants": _rows(27 * scale, 7), "eps_solve_fp64": _rows(9 * scale, 11),
                       "programs": {"a": {"runs": _rows(8 * scale, 7)}}, "paper_workloads": _rows(6 * scale, 8),
                       "peaks": {"i8": 4012.1}},
            "serving": {"req_per_s": 69695.9, "tiles": _rows(10 * scale, 3)},
            "cpu_baseline": {"value": 584.7, "per_graph": _rows(9 * scale, 8)}}


def test_line_is_short_and_whole():
    for scale in (1, 3, 40):
        full = _full(scale)
        assert len(json.dumps(full)) > 12000
        text = bench.result_line(full)
        assert "\n" not in text and len(text) <= bench.LINE_BYTES
        got = json.loads(text)
        for k, v in CONTRACT.items():
            assert got[k] == v
        assert got["left_out"] and all(isinstance(x, str) for x in got["left_out"])
    small = {**CONTRACT, "extras": {"peaks": {"i8": 4012.1}}, "per_graph": [], "serving": None, "cpu_baseline": None}
    assert json.loads(bench.result_line(small)) == small


def test_tables_are_written_by_columns():
    rows = _rows(3, 2)
    got = bench.columnar({"a": rows, "b": [1, 2], "c": [{"x": 1}, {"y": 2}]})
    assert got["a"] == {"columns": ["some_quantity_0", "some_quantity_1"], "rows": [list(r.values()) for r in rows]}
    assert got["b"] == [1, 2] and got["c"] == [{"x": 1}, {"y": 2}]
