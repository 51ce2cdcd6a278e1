"""The line bench.py prints: one JSON object that stays short whatever was measured; the rest goes to the details."""
import argparse
import json

import bench


def test_the_line_is_short_and_the_details_hold_the_rest():
    modes = {m: {"tokens_per_s_cold": 123456.789012345, "us_per_call_cold": 123.456789012345, "us_per_call_cold_median": 1.0, "us_per_call_cold_p10": 1.0,
                 "us_per_call_cold_p90": 1.0, "hbm_frac_whole_call_cold": 0.123456789012345, "plan": {f"field{i}": i for i in range(19)},
                 "kernel_us": {f"kernel {i}" * 6: 1.23456789012345 for i in range(40)}} for m in ("refresh", "reuse")}
    roofline = {k: 1.23456789012345 for k in ("achieved", "peak", "frac", "traffic", "algorithmic_bytes_per_launch", "method_flops_per_launch",
                                              "avg_launch_us", "hbm_frac", "mfma_frac")}
    result = {"workload": "w" * 120, "modes": modes, "roofline": {"bound": "hbm", "kernel": "k" * 80, "unit": "GB/s", **roofline},
              "parity": {f"measure {i}" * 4: 1.23456789012345 for i in range(7)}, "kernel_roofs_refresh": [{"x": 1.0}] * 200, "algorithmic_bytes": {},
              "cold_rotation": {}}
    order = ["cfg2", "cfg1", "cfg3", "cfg4"]
    base = {"value": 1.23456789012345, "sample": "s" * 250, "single_thread": {"workload": "w" * 60, "ms_per_call": 1.23456789012345}}
    extra = {"paper_kernel_workload_reduced_grid": [{"y": 1.0}] * 1000}
    args = argparse.Namespace(steps=20, warmup=5)
    line, details = bench.report(args, {t: result for t in order}, order, "cfg2", base, 5123.456789012345, extra)
    text = json.dumps(line)
    assert len(text) < 4096 and "\n" not in text
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
                "config", "roofline", "cpu_baseline", "parity"):
        assert key in line
    assert line["us_per_call_cold"]["cfg4"] == {"refresh": 123.46, "reuse": 123.46}
    assert len(details["other_workloads"]) == 3 and details["paper_kernel_workload_reduced_grid"] == extra["paper_kernel_workload_reduced_grid"]
