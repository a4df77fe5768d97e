"""The line that bench.py prints: every key of its contract, short enough to survive tools that keep a run's last 8 KB."""
import json

import bench


def _report():
    run = {"workload": "cfg3_mid_layer_3x3_f32_N64", "dtype": "f32", "ms": 0.123456789, "median_ms": 0.123456789, "min_ms": 0.12345, "tflops": 123.456789012,
           "peak": 157.3, "frac": 0.5123456789, "rel_err": 1.23456789e-7, "tolerance": 2e-5, "kernel": "f32 32x32x8 direct waves8 vecw rows staged border"}
    rate = {"ms": 0.123456789, "tflops": 123.456789}
    roofline = {k: 1.23456789 for k in ("achieved", "peak", "frac", "traffic", "algorithmic_bytes", "ms_median", "ms_min")}
    roofline.update(bound="mfma", unit="TFLOP/s", target_met=True, per_config=[run] * 5, achievable_peak={"f32": 156.4812345},
                    achievable_peak_random_operands={"f32": 155.512345})
    out = {"metric": "m" * 60, "value": 120.99841811782368, "unit": "TFLOP/s", "n_gpus": 1, "steps": 20, "warmup": 5, "ms_per_step": 0.11151505788167318,
           "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic (seeded)", "paper_context": "p" * 130,
           "config": {"workload": "w", "kernel": run["kernel"], "grid": 768, "parallelism": "single GPU", "workspace_bytes": 0, "clock_warmup": "c" * 200},
           "roofline": roofline, "cpu_baseline": {"value": 0.028, "unit": "TFLOP/s", "cores": 16, "kind": "oracle", "sample": "s" * 90},
           "device": {"name": "AMD Instinct MI355X", "compute_units": 256, "clock_mhz": 2400.0}, "per_config": [run] * 5, "table2_layers": [run] * 5}
    out["table2_batch_sweep"] = {"mini_batches": [16, 32, 64, 128, 256], "mean_tflops": [111.80177312996427] * 5}
    out["backward"] = [{"workload": "layer %d of a long name" % i, "backward_data": rate, "backward_filter": rate} for i in range(8)]
    out["padded_filter_layers"] = [{"shape": "N128 C96 27x27 K256 5x5 pad %d" % i, "forward": rate, "backward_data": rate} for i in range(6)]
    out["small_mini_batch_layers"] = [{"shape": "N4 C512 7x7 K512 3x3 pad %d" % i, "ms": 0.032002699375152585} for i in range(8)]
    out["other_functions"] = [{"function": "pooling 3x3 stride 2 max, backward, double precision %d" % i, "gb_per_s": 4425.45863357149} for i in range(30)]
    out["other_functions"].append({"function": "fused", "ms": 0.15})
    out["double_precision"] = [{"forward": rate, "backward_data": rate, "backward_filter": rate}] * 2
    return out


def test_line_is_short_and_complete():
    out = _report()
    line = json.dumps(bench.brief(out))
    assert len(line) < 7000, len(line)
    got = json.loads(line)
    for key in ("metric", "value", "unit", "n_gpus", "steps", "warmup", "ms_per_step", "higher_is_better", "scaling", "vs_baseline", "dtype", "data",
                "config", "roofline", "cpu_baseline"):
        assert key in got, key
    assert got["value"] == out["value"] and got["ms_per_step"] == out["ms_per_step"]
    assert len(got["roofline"]["per_config"]) == 5 and got["roofline"]["per_config"][0]["tflops"] == 123.46


def test_headline_only():
    out = _report()
    for key in ("table2_layers", "backward", "padded_filter_layers", "small_mini_batch_layers", "other_functions"):
        out[key] = []
    out["table2_batch_sweep"] = out["double_precision"] = None
    assert "other_functions_gb_per_s" not in bench.brief(out) and bench.brief(out)["value"] == out["value"]
