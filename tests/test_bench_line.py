"""The benchmark's printed line is short, whatever the side measurements add,
and nothing of the full record is lost between it and the details."""
import json
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench


def full_record():
    long = {"note": "x" * 3000, "levels": list(range(500))}
    out = {k: 1.5 for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
                            "higher_is_better", "scaling", "vs_baseline", "dtype", "data")}
    out.update({k: dict(long, value=2) for k in ("step", "kernels", "dobfs", "serving", "batched",
                                                 "sssp", "cpu_baseline")})
    out["config"] = dict(long, workload="w", rmat_n=1)
    out["roofline"] = dict(long, kernel="k", frac=0.5)
    return out


def test_line_is_short_and_whole():
    out = full_record()
    line, details = bench.split_record(out)
    assert len(json.dumps(line)) < 2000
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step",
              "higher_is_better", "scaling", "vs_baseline", "dtype", "data"):
        assert line[k] == out[k]
    assert line["config"] == {"workload": "w", "rmat_n": 1}
    assert line["roofline"] == {"kernel": "k", "frac": 0.5}
    for k, v in out.items():
        assert details.get(k, line.get(k)) == v
