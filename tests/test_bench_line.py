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


def test_rotations_count_what_can_stay_in_the_cache():
    """Inputs are read through the cache and outputs are stored past it: the inputs of a rotation have to exceed it twice."""
    from workloads import FULL_CONFIGS
    for config in ("C2", "C3", "C4", "C5"):
        bytes_in, _ = bench.traffic_split(FULL_CONFIGS[config]())
        sets = bench.rotation_sets(FULL_CONFIGS[config](), 4096)
        assert sets * bytes_in >= 2 * bench.CACHE_BYTES and (sets - 1) * bytes_in < 2 * bench.CACHE_BYTES + (64 << 20), config


def test_profiled_traffic_is_that_of_the_kernel_itself(tmp_path, monkeypatch):
    assert bench._profiled_traffic("C2", "layernorm_wave<f32,bf16,K99,L64>") is None   # a shape that no profile names
    (tmp_path / "p.md").write_text("TRAFFIC_BYTES_PER_STEP C2 layernorm_wave<f32,bf16,K3,L64> 63038332\n")
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    monkeypatch.setattr(bench, "TRAFFIC_PROFILE", "p.md")
    assert bench._profiled_traffic("C2", "layernorm_wave<f32,bf16,K3,L64>") == 63038332.0
    assert bench._profiled_traffic("C2", "layernorm_wave<f32,bf16,K6,L32>") is None
    assert bench._profiled_traffic("C3", "softmax_wave<f16,K2,L8>") is None
