"""The benchmark's line on stdout: everything that names the measurement, and short enough that a reader who keeps the last
8000 characters has it whole."""
import json

import bench


def test_the_line_holds_the_measurement_and_stays_short():
    row = bench._row({"kernel": "bias_gelu_dbias<bf16,W4,U4,RB128,fold>+colfold", "scheme": "global", "n_kernels": 2, "bytes_min": 302008320, "us": 52.123456789,
                      "GBps": 5793.123456, "frac_of_peak": 0.724, "unfused_us": 503.25, "unfused_kernels": 6, "speedup_vs_unfused": 9.654, "launches_timed": 2000,
                      "grid": 768, "block": 256, "vgprs": 116, "lds_bytes": 8196, "probe": {"mix": "2r:1w", "us": 45.8123}, "bound_us": 43.2612, "frac_of_bound": 0.8312,
                      "frac_of_probe": 0.8791, "grid_floor_us": 3.25}, "C4")
    text = "x" * 400
    result = {k: 1.234567890123456 for k in bench.LINE_KEYS}
    result.update({"metric": text, "config": {"workload": text, "kernel": row["kernel"], "grid": [768, 1, 1]}, "cpu_baseline": {"sample": text},
                   "roofline": {"bound": "hbm", "note": text, "ceilings_GBps": {str(i): 6123.123456789 for i in range(7)},
                                "per_config": {tag: dict(row) for tag, _, _ in bench.PER_CONFIG}},
                   "per_config_details": {"C1": text * 20}, "generic_patterns": {"G1": text * 20}})
    line, context = bench.split_line(result)
    assert set(line) == set(bench.LINE_KEYS) and set(context) == {"per_config_details", "generic_patterns"}
    assert len(json.dumps(line)) < 8000, len(json.dumps(line))
