"""The benchmark's result line stays short enough to be read back whole, and holds
the timed workload's entries unchanged, however many curves the record has."""
import json

import bench


def test_result_line_is_short():
    curve = [1.0 / 3.0 + q for q in range(41)]
    leg = {"value": 7.123456789e12, "ms": 1.0 / 7.0, "curve": curve, "at": [{"snr": 2.0, "gmi": 1.0 / 3.0}] * 16,
           "note": "what it is " * 20, "pair": [1.0 / 3.0, 2]}
    rec = {"metric": bench.METRIC, "value": 7.7015166928829063e12, "unit": "sample*points/s", "n_gpus": 1, "steps": 20,
           "warmup": 5, "ms_per_step": 42.547463449999953, "higher_is_better": True, "scaling": "weak",
           "vs_baseline": None, "dtype": "f32", "data": "synthetic", "config": {"snr_db": curve[:16]},
           "roofline": {"frac": 1.0 / 3.0, "traffic": None}, "gmi": curve[:16],
           **{f"leg{q}": {"a": leg, "b": leg, "c": leg} for q in range(14)}}
    assert len(json.dumps(rec)) > 20000
    line = bench.result_line(rec)
    assert len(line) <= 8000 and "\n" not in line
    out = json.loads(line)
    for k in bench.CONTRACT:
        assert out[k] == rec[k]
    assert out["leg0"]["a"] == {"value": 7.12346e12, "ms": 0.142857, "pair": [0.333333, 2]}
    assert out["gmi"] == [float(f"{v:.6g}") for v in curve[:16]]
