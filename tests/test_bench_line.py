"""bench.py prints one JSON line that fits the end of a log, with the headline
and its configuration; the legs' details stay in --detail's file."""
import json

import bench


def _leg(calls):
    rows = [{"call": f"dgrad b{i}.m0b+SiLU'", "ms": 0.1234, "bound": "hbm", "frac": 0.4321, "gbps": 4321.5,
             "tflops": 512.3, "mfma_frac": 0.0513} for i in range(calls)]
    return {"ms_per_step": 3.6, "value": 264.1, "gemm_gflop": 950.0, "calls": calls, "instep_sum_ms": 3.5,
            "ms_by_kind": {f"kind{i}": 0.25 for i in range(12)}, "roofline": {"kernel": "fwd b0", "ms": 0.2},
            "top_calls": rows[:12], "all_calls": rows, "bytes_vs_naive": {"layers": {f"b{i}": rows[0] for i in range(51)}}}


def test_line_is_short_and_whole():
    out = {"metric": "m" * 80, "value": 264.1, "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 3.6,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "d" * 60, "data": "synthetic",
           "config": {"workload": "w" * 500, "global_batch": 64}, "roofline": {"kernel": "fwd b0", "traffic": "t" * 200},
           "yolo_step": _leg(260), "latent_replay_step": dict(_leg(40), workload="w" * 400),
           "layer_sweep": {f"layer{i}": _leg(3) for i in range(20)}, "cpu_baseline": {"sample": "s" * 300}}
    full = json.dumps(out)
    line = bench.brief(out)
    assert len(full) > 30000 and len(json.dumps(line)) < 6000
    for k in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling",
              "vs_baseline", "dtype", "data", "config", "roofline", "cpu_baseline"):
        assert line[k] == out[k]
    assert json.dumps(out) == full                     # the detail is left whole
