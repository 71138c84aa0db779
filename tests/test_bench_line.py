"""bench.py's result line and its LDS bound (no GPU needed)."""
import json
import sys

from conftest import ROOT


def _bench():
    if ROOT not in sys.path:
        sys.path.insert(0, ROOT)
    import bench

    return bench


def test_result_line_is_short(capsys):
    bench = _bench()
    roof = {"kernel": "k", "bound": "hbm", "achieved": 1.23456789012, "frac": 0.1, "note": "n" * 200,
            "lds_pair_loop": {"bound_ms": 1.0, "note": "n" * 150}}
    var = {"value": 1.0e11 / 3, "ms_per_step": 1.0 / 3, "collide": roof, "stream": roof, "config": {"cells": [64, 64]}}
    line = {"metric": bench.METRIC, "value": 1.0e11 / 7, "unit": "node-updates/s", "n_gpus": 1, "steps": 100,
            "warmup": 20, "ms_per_step": 6.5 / 3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
            "dtype": "f32", "data": "synthetic", "config": {"workload": "w" * 80, "cells": [200, 200]},
            "roofline": roof, "kernels": {"stream": roof}, "cpu_baseline": {"value": 4.4e7, "sample": "s" * 300},
            "variants": dict({"v%d" % i: var for i in range(8)},
                             full_length={k: dict(var, D_trace={"t": list(range(50))}) for k in ("a", "b")},
                             adjoint={"ms_per_adjoint_step": 0.8, "window": {"steps": 200}},
                             batch={"graph": var, "tuned": {"classes": [var] * 3}})}
    bench._json_line(line)
    out = capsys.readouterr().out.strip().split("\n")
    assert len(out) == 2 and not out[0].startswith("{")
    got = json.loads(out[1])
    assert len(out[1]) < 4000
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert k in got
    assert set(got["variants"]["v0"]) == {"value", "ms_per_step"}
    assert json.loads(out[0][len("[bench] record "):])["variants"]["batch"]["tuned"]


def test_lds_bound_counts_grouped_records():
    bench = _bench()
    a, b = bench._lds_pair_bound(1e8, 1e-3), bench._lds_pair_bound(1e8, 1e-3, True)
    assert abs(b["bound_ms"] / a["bound_ms"] - (1.25 / 9.4 + 3.25 / 4.43) / (2 / 9.4 + 4 / 4.43)) < 1e-12
    assert bench.records_grouped("fixed", 4096, 20000, 8000, 0)
    assert not bench.records_grouped("fixed", 1024, 20000, 8000, 0)
    assert bench.records_grouped("part", 40000, 50000, 13824, 0)
    assert not bench.records_grouped("fixed", 4096, 20000, 8000, 64)
    assert not bench.records_grouped("hybrid", 40000, 50000, 13824, 0)
