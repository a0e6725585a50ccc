"""The benchmark's line (host logic): the lists of per-job accuracy records, some
50 KB, stay out of it and go to the file of --records; what stays is rounded,
and fits a reader of 8,000 characters."""
import json
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench


def test_records_leave_the_line():
    rec = {"job": 1, "fp32v": {"rel_dE0": 1e-9}}
    out = {"metric": "m", "value": 1.0, "config": {"dim": 3},
           "batched": {"engine_fp64": {"s": 1.0}, "vs_oracle": {"summary": {"jobs": 80}, "per_job": [rec] * 80}},
           "serving": {"rates": [{"x_R1": 1.0}], "vs_oracle": {"summary": {}, "per_request": [rec] * 50}}}
    line, recs = bench.split_records(out)
    assert recs == {"batched": {"vs_oracle": {"per_job": [rec] * 80}}, "serving": {"vs_oracle": {"per_request": [rec] * 50}}}
    assert line == {"metric": "m", "value": 1.0, "config": {"dim": 3},
                    "batched": {"engine_fp64": {"s": 1.0}, "vs_oracle": {"summary": {"jobs": 80}}},
                    "serving": {"rates": [{"x_R1": 1.0}], "vs_oracle": {"summary": {}}}}
    assert len(json.dumps(line)) < 400 < len(json.dumps(out)) // 10


def test_a_line_without_records_is_unchanged():
    out = {"metric": "m", "value": 2.5, "config": {"a": [1, 2]}, "vs_baseline": None}
    assert bench.split_records(out) == (out, {})


def test_the_line_fits_and_keeps_the_headline():
    rec = {"job": 1, "fp32v": {"rel_dE0": 1.0 / 3}}
    head = {"metric": "m", "value": 1084.123456789, "unit": "GB/s", "ms_per_step": 2.4449, "config": {"dim": 165636900},
            "roofline": {"frac": 0.13551234}}
    out = dict(head, batched={"s": 1 / 3, "e0": -70.808414466442123, "vs_oracle": {"per_job": [rec] * 400}},
               serving={"rates": [{"x": i / 7} for i in range(100)]}, big={"a": ["x" * 50] * 300})
    text, recs = bench.bench_line(out)
    line = json.loads(text)
    assert len(text) < 8000 and "\n" not in text
    assert all(line[k] == out[k] for k in ("metric", "value", "unit", "ms_per_step", "config"))
    assert line["batched"]["s"] == 0.333333 and line["batched"]["e0"] == -70.80841446644
    assert recs["batched"] == {"vs_oracle": {"per_job": [rec] * 400}}
    assert recs["big"] == out["big"] and line["big"] == "in the file of --records" and len(line["serving"]["rates"]) == 100
